// Where the tokens of a chunk sit (paper Sec. 1: a sequence of L tokens is cut into ceil(L / C)
// chunks of at most C tokens).  Two layouts:
//   fixed   B sequences of Tlen tokens each, token t of sequence b at row b * Tlen + t;
//           chunk id bc = b * cps + k, cps = ceil(Tlen / C);
//   varlen  sequences packed back to back; cu_seqlens[s] = first token row of sequence s,
//           cu_chunks[s] = id of its first chunk (both device arrays of n_seq + 1 entries);
//   packed  the same by the sequences' lengths alone, which travel with the kernel's arguments (KernelMap).
// A last chunk with fewer than C tokens is treated as padded with tokens whose key and beta are
// zero: the padded rows and columns of A vanish and T has identity rows and columns there.
#pragma once
#include <stdint.h>
#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#define TRIINV_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define TRIINV_HOST_DEVICE inline  // plain C++: the map is host-testable
#endif

namespace triinv {

struct ChunkMap {
    int64_t Tlen;               // fixed layout: tokens per sequence; varlen, packed: total number of tokens
    uint32_t cps;               // fixed layout: chunks per sequence, else 0
    uint32_t n_seq;             // varlen, packed: number of sequences
    const int64_t* cu_seqlens;  // varlen (device), else null
    const int64_t* cu_chunks;   // varlen (device), else null
    const int64_t* lens = nullptr;  // packed (host memory; the kernels get its values), else null
};

// The map as a kernel's argument.  Packed: up to 64 lengths, a lane of a wavefront each, in as many bits as the longest needs, as far as they fit
// WORDS words; the sum of the lengths and their number of chunks are known to be right (the host has checked them).  The storing kernels have
// 12 words, which leaves their arguments at 104 bytes: with 128 and more a small call took the host 0.14 us longer (4.54 us -> 4.69) whether
// it used them or not.  The kernels that apply the inverse to one right-hand side are beyond that anyhow and have 24.  Against offsets in memory,
// which a kernel of their own writes first, a call of 48 sequences of 5 tokens takes 5.1 us instead of 9.4, one of 3540 matrices 35.8 instead of 38.8.
constexpr int MAX_PACKED_SEQS = 64, MAX_PACKED_BITS = 24;

template <int WORDS> struct KernelMap {
    static_assert(WORDS >= 6 && WORDS % 2 == 0, "in place of the other fields");
    static constexpr uint32_t PACKED = 0x80000000u;
    uint32_t cps, n_seq;  // cps, packed: PACKED | bits of a length
    union {
        struct {
            int64_t Tlen;
            const int64_t *cu_seqlens, *cu_chunks;  // (addresses as such: made of integers they are no longer known to be of device memory)
        };
        uint32_t w[WORDS];  // packed
    };

    KernelMap() = default;
    explicit KernelMap(const ChunkMap& m) : cps(m.cps), n_seq(m.n_seq), w{}
    {
        if (!m.lens) {
            Tlen = m.Tlen, cu_seqlens = m.cu_seqlens, cu_chunks = m.cu_chunks;
            return;
        }
        const int bits = bits_of(m.lens, (int)m.n_seq);
        cps = PACKED | (uint32_t)bits;
        for (int s = 0; s < (int)m.n_seq; ++s) {
            const uint64_t x = (uint64_t)m.lens[s] << (s * bits & 31);
            w[s * bits >> 5] |= (uint32_t)x;
            if (x >> 32) w[(s * bits >> 5) + 1] |= (uint32_t)(x >> 32);
        }
    }
    // Bits of the longest, or 0 where these lengths do not go with the arguments.
    static int bits_of(const int64_t* lens, int n)
    {
        if (!lens || n < 1 || n > MAX_PACKED_SEQS) return 0;
        int64_t any = 1;
        for (int s = 0; s < n; ++s) {
            if (lens[s] < 0 || lens[s] >> MAX_PACKED_BITS) return 0;
            any |= lens[s];
        }
        const int bits = 64 - __builtin_clzll((unsigned long long)any);
        return bits * n <= 32 * WORDS ? bits : 0;
    }
    // Whether a kernel with this argument can be told where the tokens of m are (launch_kernel asks every one).
    static bool takes(const ChunkMap& m) { return !m.lens || bits_of(m.lens, (int)m.n_seq) > 0; }
    TRIINV_HOST_DEVICE bool packed() const { return cps & PACKED; }
    TRIINV_HOST_DEVICE uint32_t length(uint32_t s) const
    {
        const uint32_t bits = cps & ~PACKED, at = s * bits, i = at >> 5 < WORDS - 2 ? at >> 5 : WORDS - 2;
        const uint64_t two = (uint64_t)w[i + 1] << 32 | w[i];
        return s < n_seq ? (uint32_t)(two >> ((at - 32 * i) & 63)) & ((1u << bits) - 1) : 0u;
    }
    TRIINV_HOST_DEVICE ChunkMap plain() const { return ChunkMap{Tlen, cps, n_seq, cu_seqlens, cu_chunks}; }
};
// The argument of kernels that are never given lengths.
struct OffsetMap {
    int64_t Tlen;
    uint32_t cps, n_seq;
    const int64_t *cu_seqlens, *cu_chunks;
    static bool takes(const ChunkMap& m) { return !m.lens; }
    OffsetMap() = default;
    explicit OffsetMap(const ChunkMap& m) : Tlen(m.Tlen), cps(m.cps), n_seq(m.n_seq), cu_seqlens(m.cu_seqlens), cu_chunks(m.cu_chunks) {}
};

template <bool PACKED, int WORDS> struct ArgumentMap {
    typedef KernelMap<WORDS> type;
};
template <int WORDS> struct ArgumentMap<false, WORDS> {
    typedef OffsetMap type;
};
typedef KernelMap<12> InvMap;
template <bool PACKED> using InvMapIf = typename ArgumentMap<PACKED, 12>::type;
template <bool PACKED> using SolveMap = typename ArgumentMap<PACKED, 24>::type;

struct ChunkPos {
    int64_t tok0;  // row of the chunk's first token
    int valid;     // its number of tokens, 1..C
};

#if defined(__HIP_DEVICE_COMPILE__)
// At a kernel's start: its arguments loaded at once, before n_chunk, which is used first.  Left to where they are used, behind one branch of the map
// after the other, they are four loads of which each waits for the last.  (Not volatile: that would count as a write to memory, and what is
// read behind it would not go through the scalar cache.)
template <class N, class Map>
__device__ __forceinline__ void arguments_together(N& n_chunk, const void* a, const void* b, const void* c, const void* d, const Map& m)
{
    asm("" : "+s"(n_chunk) : "s"(a), "s"(b), "s"(c), "s"(d), "s"(m.cps), "s"(m.n_seq), "s"(m.Tlen), "s"(m.cu_seqlens));
}
// Sum of x over the lanes up to this one.
__device__ __forceinline__ uint32_t lane_sums(uint32_t x)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1, 2, 4, 8: within rows of 16 lanes
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1 and 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2 and 3
    return x;
}
#elif defined(__HIPCC__)
template <class N, class Map> __device__ __forceinline__ void arguments_together(N&, const void*, const void*, const void*, const void*, const Map&) {}
#endif

// The offset arrays of the varlen layout are trusted but not believed: whatever they hold (a chunk id at or beyond
// cu_chunks[n_seq], offsets that disagree with each other, trailing empty sequences), the returned first token lies
// inside [first token of the sequence found, its last token] and inside [0, total tokens - 1], and valid >= 1, so every
// row a kernel reads afterwards (tok0 .. tok0 + valid - 1) is a row of the caller's buffers.
template <int C> TRIINV_HOST_DEVICE ChunkPos locate_chunk(const ChunkMap& map, uint32_t bc)
{
    ChunkPos p;
    int64_t left;
    if (__builtin_expect(map.cu_seqlens == nullptr, 1)) {
        const uint32_t s = bc / map.cps, k = bc - s * map.cps;
        p.tok0 = (int64_t)s * map.Tlen + (int64_t)k * C;
        left = map.Tlen - (int64_t)k * C;
    } else {
        // the sequence s with cu_chunks[s] <= bc < cu_chunks[s + 1]; at most 32 halvings
        uint32_t lo = 0, hi = map.n_seq;
        for (int it = 0; it < 32 && hi - lo > 1; ++it) {
            const uint32_t mid = lo + (hi - lo) / 2;
            if (map.cu_chunks[mid] <= (int64_t)bc) lo = mid; else hi = mid;
        }
        const int64_t total = map.Tlen;
        int64_t first = map.cu_seqlens[lo], end = map.cu_seqlens[lo + 1];  // tokens [first, end) of the sequence
        if (end > total) end = total;
        if (first > end - 1) first = end - 1;
        if (first < 0) first = 0;
        int64_t tok0 = first + ((int64_t)bc - map.cu_chunks[lo]) * C;
        if (tok0 > end - 1) tok0 = end - 1;
        if (tok0 < first) tok0 = first;
        p.tok0 = tok0;
        left = end - tok0;
    }
    p.valid = left >= C ? C : (left < 1 ? 1 : (int)left);
    return p;
}

template <int C, int WORDS> TRIINV_HOST_DEVICE ChunkPos locate_packed(const KernelMap<WORDS>& map, uint32_t bc)
{
    // chunk k of the sequence found, whose tokens are first .. first + len - 1
    uint32_t first, len, k, total;
#if defined(__HIP_DEVICE_COMPILE__)
    // Every lane one sequence: running sums of tokens and chunks over the lanes, then the first sequence whose chunks end beyond bc.
    // All 64 lanes are active and agree on bc.
    len = map.length(__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)));
    const uint32_t chunks = (len + C - 1) / C, end = lane_sums(len), chunk_end = lane_sums(chunks);
    const uint64_t beyond = __builtin_amdgcn_ballot_w64(chunk_end > bc);
    const int s = beyond ? __builtin_ctzll(beyond) : MAX_PACKED_SEQS - 1;
    total = __builtin_amdgcn_readlane(end, MAX_PACKED_SEQS - 1);
    first = __builtin_amdgcn_readlane(end - len, s);
    k = bc - __builtin_amdgcn_readlane(chunk_end - chunks, s);
    len = __builtin_amdgcn_readlane(len, s);
#else
    uint32_t s = 0;
    first = 0, k = bc, len = map.length(0);
    while (s + 1 < (uint32_t)MAX_PACKED_SEQS && k >= (len + C - 1) / C) {
        first += len;
        k -= (len + C - 1) / C;
        len = map.length(++s);
    }
    total = first + len;
#endif
    const int64_t left = (int64_t)len - (int64_t)k * C;
    if (left < 1) return ChunkPos{(int64_t)total - 1, 1};  // (a chunk id beyond the last)
    return ChunkPos{(int64_t)first + (int64_t)k * C, left >= C ? C : (int)left};
}

template <int C, int WORDS> TRIINV_HOST_DEVICE ChunkPos locate_chunk(const KernelMap<WORDS>& map, uint32_t bc)
{
    return __builtin_expect(map.packed(), 0) ? locate_packed<C>(map, bc) : locate_chunk<C>(map.plain(), bc);
}
template <int C> TRIINV_HOST_DEVICE ChunkPos locate_chunk(const OffsetMap& map, uint32_t bc)
{
    return locate_chunk<C>(ChunkMap{map.Tlen, map.cps, map.n_seq, map.cu_seqlens, map.cu_chunks}, bc);
}

}  // namespace triinv
