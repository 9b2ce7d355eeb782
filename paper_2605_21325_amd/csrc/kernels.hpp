// Kernels.  One 64-lane wavefront inverts one chunk matrix (C = 16 * NB) entirely in registers:
//   k_tri_inv             A given in global memory                          -> T
//   k_gdn_tri_inv         K, beta, g -> Gram on the matrix cores, scalar gate -> T   (A never leaves the registers;
//                         four wavefronts = four adjacent heads per workgroup at C <= 64)
//   k_kda_tri_inv         per-channel gate: gated keys contracted 32 channels at a time
//   k_gdn_any_dk_tri_inv  head dimensions without a specialised build (channel loop)
//   k_tri_inv_fwd_shuffle64  row-by-row forward substitution with wavefront shuffles (baseline variant)
// and, at C = 128, four wavefronts per matrix with tiles in LDS for the methods whose state does not fit
// one wavefront: k_*_neumann128 (Neumann product), k_*_ns128 (Newton-Schulz; eight with few matrices).
// With few matrices the recursions have kernels that spread one over four or eight wavefronts: team64.hpp, team128.hpp.
// Methods: forward substitution (fp32, 16 rows at a time), blocked recursion, mixed
// recursion, blocked recursion from directly solved blocks, Neumann product, Newton-Schulz, refinement
// (inv_core.hpp).  csrc/chunk_map.hpp says where a chunk's tokens are.
#pragma once
#include "chunk_map.hpp"
#include "dispatch.hpp"
#include "inv_core.hpp"

namespace triinv {

enum : int { M_FWD = 0, M_BLOCK = 1, M_NEUMANN = 2, M_MIXED = 3, M_BLOCK_DIRECT = 4, M_NEWTON_SCHULZ = 5, M_MIXED32 = 6,
             M_BUILD_A = 100 /* no inversion: the chunk matrix A itself is written (not a triinv_method) */ };
static_assert(M_FWD == TRIINV_FWD_SUBST && M_BLOCK == TRIINV_BLOCK_RECURSIVE && M_NEUMANN == TRIINV_NEUMANN && M_MIXED == TRIINV_MIXED &&
                  M_BLOCK_DIRECT == TRIINV_BLOCK_DIRECT && M_NEWTON_SCHULZ == TRIINV_NEWTON_SCHULZ && M_MIXED32 == TRIINV_MIXED_B32,
              "the numbers of triinv_method");
enum : int { G_SCALAR = 0, G_CHANNEL = 1, G_NONE = 2 };

__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------------------------------------
// Tile source 1: A in global memory (row-major C x C, element type IN), a load per tile.
// ---------------------------------------------------------------------------------------------
template <int IN> __device__ __forceinline__ float widen16(uint16_t u) { return IN == OP_F16 ? f16_to_f32(u) : bf16_to_f32(u); }

template <int NB, int IN> struct GlobalA {
    static constexpr int C = 16 * NB;
    static constexpr bool kFromMemory = true;   // a tile is a plain load: fetch it when it is needed
    static constexpr bool kHoldsKeys = false;
    const void* base;  // first element of this matrix
    Lane ln;

    template <bool TR> __device__ __forceinline__ v4f get(int i, int j) const
    {
        v4f v;
        if (!TR) {  // v[r] = A[16i + 4q + r][16j + n]
            const int off = (16 * i + 4 * ln.q) * C + 16 * j + ln.n;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if constexpr (IN == OP_F32)
                    v[r] = static_cast<const float*>(base)[off + r * C];
                else
                    v[r] = widen16<IN>(static_cast<const uint16_t*>(base)[off + r * C]);
            }
            if (i == j) {
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = (4 * ln.q + r > ln.n) ? v[r] : 0.f;
            }
        } else {  // v[r] = A[16i + n][16j + 4q + r]
            const int off = (16 * i + ln.n) * C + 16 * j + 4 * ln.q;
            if constexpr (IN == OP_F32) {
                v = *reinterpret_cast<const v4f*>(static_cast<const float*>(base) + off);
            } else {
                const v2u u = *reinterpret_cast<const v2u*>(static_cast<const uint16_t*>(base) + off);
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = widen16<IN>((uint16_t)(r & 1 ? u[r / 2] >> 16 : u[r / 2] & 0xffff));
            }
            if (i == j) {
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = (ln.n > 4 * ln.q + r) ? v[r] : 0.f;
            }
        }
        return v;
    }
};

// The same with the element type known at run time only, for kernels that read most tiles twice (fp32 A; for a 16-bit one see
// LoadedA16).  Each tile is then loaded in a block of its own, behind a branch that the whole wavefront takes: the
// compiler can neither move all loads to the start, where they cost the Neumann product a wavefront per SIMD, nor put off a second
// reading until the tile has left the caches.  (Scheduling fences between typed loads: 533 and 210 us where this takes 460 and 161.)
template <int NB> struct GlobalAnyA {
    static constexpr bool kFromMemory = true;
    static constexpr bool kHoldsKeys = false;
    const void* base;
    int dt;
    Lane ln;
    template <bool TR> __device__ __forceinline__ v4f get(int i, int j) const
    {
        constexpr int C = 16 * NB;
        const int64_t off = TR ? (int64_t)(16 * i + ln.n) * C + 16 * j + 4 * ln.q : (int64_t)(16 * i + 4 * ln.q) * C + 16 * j + ln.n;
        v4f v;
        if (dt == OP_F32) {
            const float* const p = static_cast<const float*>(base) + off;
            if constexpr (TR) {
                v = *reinterpret_cast<const v4f*>(p);
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = p[r * C];
            }
        } else {
            const uint16_t* const p = static_cast<const uint16_t*>(base) + off;
            uint16_t u[4];
            if constexpr (TR) {
                const v2u w = *reinterpret_cast<const v2u*>(p);
#pragma unroll
                for (int r = 0; r < 4; ++r) u[r] = (uint16_t)(r & 1 ? w[r / 2] >> 16 : w[r / 2] & 0xffff);
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) u[r] = p[r * C];
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = dt == OP_F16 ? f16_to_f32(u[r]) : bf16_to_f32(u[r]);
        }
        if (i == j) {
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = (TR ? ln.n > 4 * ln.q + r : 4 * ln.q + r > ln.n) ? v[r] : 0.f;
        }
        return v;
    }
};

// ---------------------------------------------------------------------------------------------
// Tile source 2: A built from the keys.  S = K_c K_c^T on the matrix cores with the stored key
// values as operands (16x16x32 for 16-bit keys, 16x16x4 for fp32 keys), then
// A_ij = beta_i exp(g_i - g_j) S_ij in fp32 (paper Table 1, GDN / DeltaNet rows).
// KD: storage type of K.  DKS: number of k-steps (32 channels each for 16-bit keys, 16 for fp32).
// ---------------------------------------------------------------------------------------------
template <int KD> struct KeyVec;
template <> struct KeyVec<OP_F32> { typedef v4f type; };
template <> struct KeyVec<OP_F16> { typedef v8h type; };
template <> struct KeyVec<OP_BF16> { typedef v8bf type; };

template <int KD> __device__ __forceinline__ v4f gram_step(typename KeyVec<KD>::type a, typename KeyVec<KD>::type b, v4f acc);
template <> __device__ __forceinline__ v4f gram_step<OP_F32>(v4f a, v4f b, v4f acc)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[r], b[r], acc, 0, 0, 0);
    return acc;
}
template <> __device__ __forceinline__ v4f gram_step<OP_F16>(v8h a, v8h b, v4f acc)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, acc, 0, 0, 0);
}
template <> __device__ __forceinline__ v4f gram_step<OP_BF16>(v8bf a, v8bf b, v4f acc)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
}

// beta / g of one chunk's tokens in the two index patterns a lane needs (by its column n, by its
// rows 4q + r), and the scalar gate applied to a Gram tile:
//   A_ij = beta_i exp(g_i - g_j) S_ij for i > j, else 0      (paper Table 1, GDN / DeltaNet rows).
// g is kept multiplied by log2(e) (done once per token when the values are staged), so that the gate of an element is
// one subtraction and one exp2; without a gate g = 0 and exp2(0) = 1 exactly, so that kind needs no code of its own.
// NOGATE: the launch is known to have no gate (gc null): the factor exp(g_i - g_j) is 1 and its exponentials are left out.
template <int NB, bool NOGATE = false> struct GateVec {
    static constexpr int C = 16 * NB;
    float beta_n[NB], g_n[NB];   // g_*: g log2(e)
    v4f beta_q[NB], g_q[NB];
    bool gated;

    // Loading is split in two so that the caller can put its other global loads between the halves:
    // issue() starts the loads of this lane's beta / g values (C / 64 tokens per lane) and stage()
    // redistributes them through LDS into the two index patterns.  Vector-memory loads return in
    // order, so issuing these first lets stage() wait for them alone while later loads stay in flight.
    // bc, gc: first element of (chunk row 0, this head); tok_stride in elements; gc may be null.
    static constexpr int RAW = C >= 64 ? C / 64 : 1;
    float raw_b[RAW], raw_g[RAW];

    // valid: number of tokens the chunk really has; the rows beyond read the last real token (a valid
    // address, and a g that keeps every exponent of the gate <= 0) and get beta = 0.
    __device__ __forceinline__ void issue(const float* bc, const float* gc, int64_t tok_stride, Lane ln, int valid = C)
    {
        const int l = 16 * ln.q + ln.n;
        gated = (gc != nullptr);
        const float* gp = gated ? gc : bc;  // always a valid address: the load is unconditional, the value is not
#pragma unroll
        for (int k = 0; k < RAW; ++k) {
            const int t = l + 64 * k;
            if (C < 64 && t >= C) {  // more lanes than tokens
                raw_b[k] = 0.f;
                raw_g[k] = 0.f;
                continue;
            }
            const int tc = t < valid ? t : valid - 1;
            const float b = bc[tc * tok_stride];
            raw_b[k] = t < valid ? b : 0.f;
            raw_g[k] = gp[tc * tok_stride];
        }
    }

    // lds: wave-private, 2 * C floats.
    __device__ __forceinline__ void stage(float* lds, Lane ln)
    {
        const int l = 16 * ln.q + ln.n;
#pragma unroll
        for (int k = 0; k < RAW; ++k) {
            if (C < 64 && l >= C) continue;
            lds[l + 64 * k] = raw_b[k];
            lds[C + l + 64 * k] = gated ? raw_g[k] * 1.44269504088896340736f : 0.f;
        }
        wave_lds_sync();
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            beta_n[i] = lds[16 * i + ln.n];
            g_n[i] = lds[C + 16 * i + ln.n];
            beta_q[i] = *reinterpret_cast<const v4f*>(&lds[16 * i + 4 * ln.q]);
            g_q[i] = *reinterpret_cast<const v4f*>(&lds[C + 16 * i + 4 * ln.q]);
        }
        wave_lds_sync();
    }

    __device__ __forceinline__ void load(const float* bc, const float* gc, int64_t tok_stride, float* lds, Lane ln, int valid = C)
    {
        issue(bc, gc, tok_stride, ln, valid);
        stage(lds, ln);
    }

    // s: Gram tile (i, j) in N (TR = false) or T orientation.
    template <bool TR> __device__ __forceinline__ v4f apply(int i, int j, v4f s, Lane ln) const
    {
        v4f a;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            // N: element (row 16i + 4q + r, col 16j + n);  T: element (row 16i + n, col 16j + 4q + r)
            const float b = TR ? beta_n[i] : beta_q[i][r];
            const float d = TR ? (g_n[i] - g_q[j][r]) : (g_q[i][r] - g_n[j]);  // (g_i - g_j) log2 e
            const float w = NOGATE ? b : b * __builtin_amdgcn_exp2f(d);        // beta_i exp(g_i - g_j)
            const bool low = (i != j) || (TR ? (ln.n > 4 * ln.q + r) : (4 * ln.q + r > ln.n));
            a[r] = low ? w * s[r] : 0.f;
        }
        return a;
    }
};

template <int KD, int NB, int DKS> struct GramA {
    static constexpr bool kFromMemory = false;  // a tile costs matrix-core work and pins the key registers
    static constexpr bool kHoldsKeys = true;
    typedef typename KeyVec<KD>::type kvec;
    static constexpr int C = 16 * NB;
    static constexpr int KSTEP = (KD == OP_F32) ? 16 : 32;  // channels per k-step
    kvec k[NB][DKS];
    GateVec<NB> gate;
    Lane ln;

    // Kc: first key element of (chunk row 0, this head); row_stride in elements.
    // valid: number of tokens the chunk really has; rows beyond it read the last real token (a valid
    // address) and are then replaced by zero keys.
    __device__ __forceinline__ void load_keys(const void* Kc, int64_t row_stride, int valid = C)
    {
        constexpr int per_lane = (KD == OP_F32) ? 4 : 8;
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int s = 0; s < DKS; ++s) {
                const int row = 16 * i + ln.n;
                const int64_t off = (int64_t)(row < valid ? row : valid - 1) * row_stride + KSTEP * s + per_lane * ln.q;
                // plain loads: the non-temporal hint measured ~5 % slower here
                if (KD == OP_F32)
                    k[i][s] = *reinterpret_cast<const kvec*>(static_cast<const float*>(Kc) + off);
                else
                    k[i][s] = *reinterpret_cast<const kvec*>(static_cast<const uint16_t*>(Kc) + off);
            }
        if (valid < C) {  // wave-uniform: only a sequence's last chunk comes here
            const kvec zero = __builtin_bit_cast(kvec, v4u{0u, 0u, 0u, 0u});
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int s = 0; s < DKS; ++s)
                    if (16 * i + ln.n >= valid) k[i][s] = zero;
        }
    }

    __device__ __forceinline__ void issue_gate(const float* bc, const float* gc, int64_t tok_stride, int valid = C)
    {
        gate.issue(bc, gc, tok_stride, ln, valid);
    }
    __device__ __forceinline__ void stage_gate(float* lds) { gate.stage(lds, ln); }

    template <bool TR> __device__ __forceinline__ v4f get(int i, int j) const
    {
        v4f s = zero4();
#pragma unroll
        for (int t = 0; t < DKS; ++t) s = TR ? gram_step<KD>(k[j][t], k[i][t], s) : gram_step<KD>(k[i][t], k[j][t], s);
        return gate.template apply<TR>(i, j, s, ln);
    }
};

// ---------------------------------------------------------------------------------------------
// Which tiles of A, in which orientation, a method asks for (used by sources that have to form
// every tile up front).  The blocked recursion wants an off-diagonal tile in the orientation
// opposite to that of the merge that consumes it; that merge belongs to the smallest aligned
// block pair containing tile rows i and j.
// ---------------------------------------------------------------------------------------------
constexpr bool ROOT_T = true;  // the last merge of the blocked recursion is produced in T orientation

template <int NB> __host__ __device__ constexpr bool merge_block_is_T(int i, int j)
{
    int h = 1;
    while ((i / (2 * h)) != (j / (2 * h))) h *= 2;
    return (2 * h == NB) ? ROOT_T : (((i / (2 * h)) & 1) != 0);
}

constexpr int WITH_REFINE = 1000;  // METHOD + WITH_REFINE: the tiles of METHOD plus every tile in N orientation (Alg. 6's Y A)

template <int NB, int METHOD> __host__ __device__ constexpr bool need_tile(int i, int j, bool tr)
{
    if constexpr (METHOD >= WITH_REFINE) return !tr || need_tile<NB, METHOD - WITH_REFINE>(i, j, tr);
    if (METHOD == M_FWD || METHOD == M_NEWTON_SCHULZ || METHOD == M_BUILD_A) return tr;
    if (METHOD == M_NEUMANN) return true;
    if (METHOD == M_MIXED32 && i / 2 == j / 2) return true;  // the 32 x 32 Neumann blocks want both orientations
    if (i == j) return METHOD == M_BLOCK_DIRECT ? tr : true;
    return merge_block_is_T<NB>(i, j) ? !tr : tr;
}

// Tile source 3: all tiles precomputed in registers.
template <int NB> struct PreA {
    static constexpr bool kFromMemory = false;
    static constexpr bool kHoldsKeys = false;
    v4f n[NB * (NB + 1) / 2], t[NB * (NB + 1) / 2];
    template <bool TR> __device__ __forceinline__ v4f get(int i, int j) const { return TR ? t[tix(i, j)] : n[tix(i, j)]; }
};

// ---------------------------------------------------------------------------------------------
// Tile source 4: every tile of a given A requested before the first is used, so that a wavefront waits for memory once and not
// at every level of the recursion (fp32, where the tile-wise loads already are whole 64-byte pieces: 1-4 % at C >= 64, 8 % at
// C <= 32).
// ---------------------------------------------------------------------------------------------
template <int NB, int METHOD> struct LoadedA {  // fp32 elements
    static constexpr bool kFromMemory = true;
    static constexpr bool kHoldsKeys = false;
    PreA<NB> tiles;
    __device__ __forceinline__ void load(const void* base, Lane ln)
    {
        const GlobalA<NB, OP_F32> mem{base, ln};
#pragma unroll
        for (int d = 0; d < NB; ++d)  // in the order of use: near the diagonal first
#pragma unroll
            for (int i = d; i < NB; ++i) {
                const int j = i - d;
                if (need_tile<NB, METHOD>(i, j, true)) tiles.t[tix(i, j)] = mem.template get<true>(i, j);
                if (need_tile<NB, METHOD>(i, j, false)) tiles.n[tix(i, j)] = mem.template get<false>(i, j);
            }
    }
    template <bool TR> __device__ __forceinline__ v4f get(int i, int j) const { return tiles.template get<TR>(i, j); }
};

// 16-bit elements.  A lane loads 16 bytes of a row, two lane groups' share of a tile: two swaps between the lane groups per
// register pair (v_permlane16_swap, v_permlane32_swap) make T-orientation tiles of two neighbours out of them, which are
// matrix-core operands as they stand.  The N orientation is a product with the identity, exact for finite values (an infinity or
// NaN makes its row of the tile NaN, as the products it goes into would).  Loaded tile by tile (8 bytes a lane, 2 bytes in N
// orientation, 32-byte row pieces, each level of the recursion waiting for its own) the same kernels took: bf16 A, blocked
// recursion, 8192 matrices of C = 128, bf16 result 137 against 87 us, fp32 result 178 against 137; 16384 of C = 64, bf16 result
// 56 against 47, fp32 77 against 71; C = 16 18.2 against 11.3.
template <int IN, int OP, int NB> struct LoadedA16 {
    static constexpr int C = 16 * NB;
    static constexpr bool kFromMemory = true;
    static constexpr bool kHoldsKeys = false;
    v2u raw[NB * (NB + 1) / 2];  // T orientation
    Opnd<IN> id;

    __device__ __forceinline__ void load(const void* base, Lane ln)
    {
        const uint16_t* const p = static_cast<const uint16_t*>(base) + ln.n * C;
        if constexpr (NB == 1) {
            raw[0] = *reinterpret_cast<const v2u*>(p + 4 * ln.q);
        } else {
            v4u u[NB][(NB + 1) / 2];
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int k = 0; k <= i / 2; ++k) u[i][k] = *reinterpret_cast<const v4u*>(p + 16 * i * C + 32 * k + 8 * ln.q);
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int k = 0; k <= i / 2; ++k)
#pragma unroll
                    for (int w = 0; w < 2; ++w) {
                        // (x: columns 8q + 2w, +1;  y: columns 8q + 4 + 2w, +1) -> columns 4q + 2w, +1 of either tile
                        const auto odd = __builtin_amdgcn_permlane16_swap(u[i][k][w], u[i][k][2 + w], false, false);
                        const auto half = __builtin_amdgcn_permlane32_swap(odd[0], odd[1], false, false);
                        raw[tix(i, 2 * k)][w] = half[0];
                        if (2 * k + 1 <= i) raw[tix(i, 2 * k + 1)][w] = half[1];
                    }
        }
        const Mask<IN> low = make_mask<IN>(ln.n > 4 * ln.q, ln.n > 4 * ln.q + 1, ln.n > 4 * ln.q + 2, ln.n > 4 * ln.q + 3);
#pragma unroll
        for (int i = 0; i < NB; ++i) raw[tix(i, i)] &= low.m;
        id = pack<IN>(identity_tile(ln));
    }
    __device__ __forceinline__ Opnd<IN> stored(int i, int j) const
    {
        Opnd<IN> o;
        o.x = __builtin_bit_cast(decltype(o.x), raw[tix(i, j)]);
        return o;
    }
    template <bool TR> __device__ __forceinline__ v4f get(int i, int j) const
    {
        if constexpr (!TR) return tn<IN>(stored(i, j), id, zero4());
        v4f v;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = widen16<IN>((uint16_t)(r & 1 ? raw[tix(i, j)][r / 2] >> 16 : raw[tix(i, j)][r / 2] & 0xffff));
        return v;
    }
    template <bool TR> __device__ __forceinline__ Opnd<OP> operand(int i, int j) const
    {
        if constexpr (TR && IN == OP)
            return stored(i, j);
        else
            return pack<OP>(get<TR>(i, j));
    }
};
template <int IN, int OP, int NB> struct PackedSource<LoadedA16<IN, OP, NB>> {
    static constexpr bool value = true;
};

// One k-step (32 channels; lane (q, n) holds channels 8q..8q+7 of row n) as a matrix-core operand.
template <int OPG> struct GOp;
template <> struct GOp<OP_F32> { float x[8]; };
template <> struct GOp<OP_F16> { v8h x; };
template <> struct GOp<OP_BF16> { v8bf x; };

template <int OPG> __device__ __forceinline__ GOp<OPG> gpack(const float (&v)[8]);
template <> __device__ __forceinline__ GOp<OP_F32> gpack<OP_F32>(const float (&v)[8])
{
    GOp<OP_F32> o;
#pragma unroll
    for (int r = 0; r < 8; ++r) o.x[r] = v[r];
    return o;
}
template <> __device__ __forceinline__ GOp<OP_F16> gpack<OP_F16>(const float (&v)[8])
{
    const v4u u = {pack2_f16(v[0], v[1]), pack2_f16(v[2], v[3]), pack2_f16(v[4], v[5]), pack2_f16(v[6], v[7])};
    return {__builtin_bit_cast(v8h, u)};
}
template <> __device__ __forceinline__ GOp<OP_BF16> gpack<OP_BF16>(const float (&v)[8])
{
    const v4u u = {pack2_bf16(v[0], v[1]), pack2_bf16(v[2], v[3]), pack2_bf16(v[4], v[5]), pack2_bf16(v[6], v[7])};
    return {__builtin_bit_cast(v8bf, u)};
}

template <int OPG> __device__ __forceinline__ v4f gstep(const GOp<OPG>& a, const GOp<OPG>& b, v4f acc);
template <> __device__ __forceinline__ v4f gstep<OP_F32>(const GOp<OP_F32>& a, const GOp<OP_F32>& b, v4f acc)
{
#pragma unroll
    for (int r = 0; r < 8; ++r) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x[r], b.x[r], acc, 0, 0, 0);
    return acc;
}
template <> __device__ __forceinline__ v4f gstep<OP_F16>(const GOp<OP_F16>& a, const GOp<OP_F16>& b, v4f acc)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a.x, b.x, acc, 0, 0, 0);
}
template <> __device__ __forceinline__ v4f gstep<OP_BF16>(const GOp<OP_BF16>& a, const GOp<OP_BF16>& b, v4f acc)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.x, b.x, acc, 0, 0, 0);
}

// Eight consecutive key channels of one row as stored (16-bit: one 16-byte load; fp32: two).
template <bool K16> struct RawKey8;
template <> struct RawKey8<true> { uint4 u; };
template <> struct RawKey8<false> { v4f a, b; };

template <bool K16> __device__ __forceinline__ RawKey8<K16> load_key8(const void* Kc, int64_t off)
{
    RawKey8<K16> o;
    if constexpr (K16) {
        o.u = *reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(Kc) + off);
    } else {
        o.a = *reinterpret_cast<const v4f*>(static_cast<const float*>(Kc) + off);
        o.b = *reinterpret_cast<const v4f*>(static_cast<const float*>(Kc) + off + 4);
    }
    return o;
}

template <bool K16> __device__ __forceinline__ void widen_key8(const RawKey8<K16>& k, bool is_f16, float (&v)[8])
{
    if constexpr (K16) {
        const uint32_t w[4] = {k.u.x, k.u.y, k.u.z, k.u.w};
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint16_t lo = (uint16_t)(w[r] & 0xffff), hi = (uint16_t)(w[r] >> 16);
            v[2 * r] = is_f16 ? f16_to_f32(lo) : bf16_to_f32(lo);
            v[2 * r + 1] = is_f16 ? f16_to_f32(hi) : bf16_to_f32(hi);
        }
    } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) { v[r] = k.a[r]; v[4 + r] = k.b[r]; }
    }
}

// Per-channel gate (paper Table 1, KDA row): A_ij = beta_i sum_c k_ic k_jc exp(g_ic - g_jc)
//   = beta_i [(K * exp(G - a)) (K * exp(a - G))^T]_ij   for any per-channel anchor a.
// C <= 64: one anchor per 16-row tile row I, a_I = the first row of that tile row of G: for a tile (I, J),
// J <= I, the left factor k_i exp(g_i - a_I) has an exponent within the decay of 16 tokens and <= 0, the
// right factor k_j exp(a_I - g_j) an exponent <= 0 for J < I and within the decay of 16 tokens for J = I
// (log-decays only fall along a chunk), so neither factor can overflow however strong the decay over the
// whole chunk is; the price is a right factor per (I, J) instead of per J, which costs one multiplication by a
// channel-only factor each (see below), not an exponential.
// C = 128 (no registers for that): a single anchor, row C/2, both factors within exp(+-half the chunk's decay).
// The gated keys are rounded to OPG and contracted on the matrix cores, 32 channels per step,
// accumulating every tile the method needs; nothing but K, G, beta is read, nothing stored.
// One iteration covers one whole 128-byte line of keys per row (64 channels of 16-bit keys, i.e.
// two k-steps, or 32 channels of fp32 keys): all of a line's key loads are issued together, so
// its second half is still cached when needed (requested one k-step apart, lines were found
// evicted in between and fetched from HBM twice).
// Kc / gc: element (chunk row 0, this head, channel 0); row_stride in elements (same for both).
//
// The C <= 64 form.  The loads of a k-step's gate rows (and, every other k-step, of the next line of keys) go out before the k-step
// ahead of them is computed: one after the other, four k-steps were four round trips to memory, most of a call of few matrices.  The
// anchor rows are rows of the chunk, the ones that lanes n = 0 load anyway, and reach the others through LDS.
// Kernel time, bf16 keys of d_k = 128, C = 64, loads in the k-step itself / a step ahead: 256 matrices 11.6 / 10.9 us, 1024 18.5 / 15.6, 16384
// 214 / 201; one right-hand side, 1024 20.6 / 17.8; fp32 operands, 1024 27.3 / 24.5, d_k = 256 30.0 / 23.8.
// ahead = false: not so, for calls that fill the chip many times over and keep fewer bytes of keys than of gates in flight this way
// (fp32 keys, fp32 operands at C = 32): fp32 keys, C = 64, gate rows ahead / not, 8192 matrices 123 / 126 us, 16384 250 / 242.  C = 16 has a
// form of its own, accumulate_gated_gram16.
constexpr int GATES_AHEAD_MATRICES = 8192;
template <int OPG, int NB, int METHOD, bool K16>
__device__ __forceinline__ void accumulate_gated_gram64(PreA<NB>& out, const void* Kc, bool is_f16, const float* gc, int64_t row_stride, int n_step,
                                                        Lane ln, int valid, float* tab, bool ahead)
{
    constexpr float LOG2E = 1.44269504088896340736f;
    constexpr int STEPS = K16 ? 2 : 1;
    constexpr bool KEYS_AHEAD = K16 && (NB == 4 || (NB == 2 && OPG != OP_F32));  // elsewhere they would cost a wavefront per SIMD
    if (KEYS_AHEAD) ahead = true;
    if (METHOD == M_NEWTON_SCHULZ + WITH_REFINE) ahead = false;                  // (which has no registers left for them)
    int rowc[NB];
    float keep[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int row = 16 * i + ln.n;
        rowc[i] = row < valid ? row : valid - 1;
        keep[i] = row < valid ? 1.f : 0.f;
    }
    const auto load_keys = [&](RawKey8<K16> (&raw)[STEPS][NB], int s) {
#pragma unroll
        for (int t = 0; t < STEPS; ++t)
#pragma unroll
            for (int i = 0; i < NB; ++i)
                if (s + t < n_step) raw[t][i] = load_key8<K16>(Kc, (int64_t)rowc[i] * row_stride + 32 * (s + t) + 8 * ln.q);
    };
    const auto load_gates = [&](v4f (&G)[NB][2], int s) {
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const float* const p = gc + (int64_t)rowc[i] * row_stride + 32 * s + 8 * ln.q;
            G[i][0] = *reinterpret_cast<const v4f*>(p);
            G[i][1] = *reinterpret_cast<const v4f*>(p + 4);
        }
    };
    // Per row group (q): the anchors of its 8 channels, then the pairs' factors (see the k-step).
    constexpr int NP = NB * (NB - 1) / 2, NE = 8 * NP;
    float* const anc = tab + ln.q * (8 * NB + NE);
    float* const fac = anc + 8 * NB;

    RawKey8<K16> raw[STEPS][NB];
    v4f G[NB][2];
    if (KEYS_AHEAD) load_keys(raw, 0);
    load_gates(G, 0);
    for (int s0 = 0; s0 < n_step; s0 += STEPS) {
#pragma unroll
        for (int t = 0; t < STEPS; ++t) {
            const int s = s0 + t;
            if (s >= n_step) break;
            if (ln.n == 0) {
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    *reinterpret_cast<v4f*>(&anc[8 * i]) = G[i][0];
                    *reinterpret_cast<v4f*>(&anc[8 * i + 4]) = G[i][1];
                }
            }
            v4f G_next[NB][2];
            RawKey8<K16> raw_next[STEPS][NB];
            if (!KEYS_AHEAD && t == 0) load_keys(raw, s);
            if (s + 1 < n_step) {
                if (KEYS_AHEAD && t == STEPS - 1) load_keys(raw_next, s + 1);
                if (ahead) load_gates(G_next, s + 1);
            }
            wave_lds_sync();
            // With e_i = (g_i - a_I) log2 e (row i, its tile row's anchor a_I), u_i = k_i 2^(e_i) is the left factor of every
            // tile in tile row I and v_j = k_j 2^(-e_j) the right factor of the diagonal tile (J, J).  The right factor of
            // tile (I, J), J < I, differs from v_j by 2^((a_I - a_J) log2 e), which depends on the channel only, not on the
            // row: those NB (NB - 1) / 2 x 32 factors are computed once per k-step by the whole wave (through LDS: the 16
            // lanes of a row group need the same; each computes a share of the table) instead
            // of once per row: 67 exponentials per lane and k-step at C = 64 instead of 112, and no subtraction or scaling
            // of the exponent per pair either.
            {
#pragma unroll
                for (int k = 0; k < (NE + 15) / 16; ++k) {
                    const int e = ln.n + 16 * k, p = e >> 3, r = e & 7;
                    if (e < NE) {  // pair p = (hi, lo), hi > lo, in the order (1,0) (2,0) (2,1) (3,0) (3,1) (3,2)
                        const int hi = p >= 3 ? 3 : (p >= 1 ? 2 : 1), lo = p - hi * (hi - 1) / 2;
                        fac[e] = __builtin_amdgcn_exp2f((anc[8 * hi + r] - anc[8 * lo + r]) * LOG2E);
                    }
                }
                wave_lds_sync();
            }
            GOp<OPG> ppi[NB];
            float v[NB][8];
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                float kv[8], u[8];
                widen_key8<K16>(raw[t][i], is_f16, kv);
                const v4f a0 = *reinterpret_cast<const v4f*>(&anc[8 * i]), a1 = *reinterpret_cast<const v4f*>(&anc[8 * i + 4]);
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    const float kk = kv[r] * keep[i];
                    const float e = (G[i][r / 4][r % 4] - (r < 4 ? a0[r] : a1[r - 4])) * LOG2E;
                    u[r] = kk * __builtin_amdgcn_exp2f(e);
                    v[i][r] = kk * __builtin_amdgcn_exp2f(-e);
                }
                ppi[i] = gpack<OPG>(u);
            }
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int j = 0; j <= i; ++j) {
                    float dn[8];
                    if (i == j) {
#pragma unroll
                        for (int r = 0; r < 8; ++r) dn[r] = v[j][r];
                    } else {
                        const int p = i * (i - 1) / 2 + j;
                        const v4f f0 = *reinterpret_cast<const v4f*>(&fac[8 * p]), f1 = *reinterpret_cast<const v4f*>(&fac[8 * p + 4]);
#pragma unroll
                        for (int r = 0; r < 8; ++r) dn[r] = v[j][r] * (r < 4 ? f0[r] : f1[r - 4]);
                    }
                    const GOp<OPG> pmj = gpack<OPG>(dn);
                    if (need_tile<NB, METHOD>(i, j, false)) out.n[tix(i, j)] = gstep<OPG>(ppi[i], pmj, out.n[tix(i, j)]);
                    if (need_tile<NB, METHOD>(i, j, true)) out.t[tix(i, j)] = gstep<OPG>(pmj, ppi[i], out.t[tix(i, j)]);
                }
            wave_lds_sync();  // (anchors and factors are rewritten by the next k-step)
            if (!ahead && s + 1 < n_step) load_gates(G_next, s + 1);
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                G[i][0] = G_next[i][0];
                G[i][1] = G_next[i][1];
                if (KEYS_AHEAD && t == STEPS - 1) {
#pragma unroll
                    for (int k = 0; k < STEPS; ++k) raw[k][i] = raw_next[k][i];
                }
            }
        }
    }
}

// C = 16: one tile row, whose only anchor every lane loads, and wavefronts enough to hide the loads of one behind the others' work (through
// LDS and a step ahead as above, 1792 matrices of d_k = 256: 11.8 us against 10.6).
template <int OPG, int METHOD, bool K16>
__device__ __forceinline__ void accumulate_gated_gram16(PreA<1>& out, const void* Kc, bool is_f16, const float* gc, int64_t row_stride, int n_step,
                                                        Lane ln, int valid)
{
    constexpr float LOG2E = 1.44269504088896340736f;
    constexpr int STEPS = K16 ? 2 : 1;
    const int64_t row = (int64_t)(ln.n < valid ? ln.n : valid - 1) * row_stride + 8 * ln.q;
    const float keep = ln.n < valid ? 1.f : 0.f;
    for (int s0 = 0; s0 < n_step; s0 += STEPS) {
        RawKey8<K16> raw[STEPS];
#pragma unroll
        for (int t = 0; t < STEPS; ++t)
            if (s0 + t < n_step) raw[t] = load_key8<K16>(Kc, row + 32 * (s0 + t));
#pragma unroll
        for (int t = 0; t < STEPS; ++t) {
            if (s0 + t >= n_step) break;
            const float *const g = gc + row + 32 * (s0 + t), *const a = gc + 8 * ln.q + 32 * (s0 + t);
            const v4f G[2] = {*reinterpret_cast<const v4f*>(g), *reinterpret_cast<const v4f*>(g + 4)};
            const v4f A[2] = {*reinterpret_cast<const v4f*>(a), *reinterpret_cast<const v4f*>(a + 4)};
            float kv[8], up[8], dn[8];
            widen_key8<K16>(raw[t], is_f16, kv);
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const float kk = kv[r] * keep;
                const float e = (G[r / 4][r % 4] - A[r / 4][r % 4]) * LOG2E;
                up[r] = kk * __builtin_amdgcn_exp2f(e);
                dn[r] = kk * __builtin_amdgcn_exp2f(-e);
            }
            const GOp<OPG> u = gpack<OPG>(up), v = gpack<OPG>(dn);
            if (need_tile<1, METHOD>(0, 0, false)) out.n[0] = gstep<OPG>(u, v, out.n[0]);
            if (need_tile<1, METHOD>(0, 0, true)) out.t[0] = gstep<OPG>(v, u, out.t[0]);
        }
    }
}

// The general form: C = 128 and, with GATED = false, no per-channel gate (the stored keys themselves are the operands, OPG = their type,
// exact products, and gc is not read): the any-d_k path of the scalar / no-gate kinds.
template <int OPG, int NB, int METHOD, bool K16, bool GATED = true>
__device__ __forceinline__ void accumulate_gated_gram(PreA<NB>& out, const void* Kc, bool is_f16, const float* gc,
                                                      int64_t row_stride, int n_step, Lane ln, int valid, float* tab = nullptr, bool ahead = true)
{
    if constexpr (GATED && NB == 1) return accumulate_gated_gram16<OPG, METHOD, K16>(out, Kc, is_f16, gc, row_stride, n_step, ln, valid);
    else if constexpr (GATED && NB <= 4) return accumulate_gated_gram64<OPG, NB, METHOD, K16>(out, Kc, is_f16, gc, row_stride, n_step, ln, valid, tab, ahead);
    constexpr int C = 16 * NB;
    [[maybe_unused]] constexpr float LOG2E = 1.44269504088896340736f;
    constexpr int STEPS = (K16 && NB <= 4) ? 2 : 1;  // C = 128 has no registers to spare for the pairing
    // rows beyond the chunk's real tokens read the last real one (valid addresses, finite exponents)
    // and contribute zero keys; the anchor is a real row too
    int rowc[NB];
    float keep[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int row = 16 * i + ln.n;
        rowc[i] = row < valid ? row : valid - 1;
        keep[i] = row < valid ? 1.f : 0.f;
    }
    const int anchor = C / 2 < valid ? C / 2 : valid - 1;
    for (int s0 = 0; s0 < n_step; s0 += STEPS) {
        RawKey8<K16> raw[STEPS][NB];
#pragma unroll
        for (int t = 0; t < STEPS; ++t)
#pragma unroll
            for (int i = 0; i < NB; ++i)
                if (s0 + t < n_step) raw[t][i] = load_key8<K16>(Kc, (int64_t)rowc[i] * row_stride + 32 * (s0 + t) + 8 * ln.q);
#pragma unroll
        for (int t = 0; t < STEPS; ++t) {
            if (s0 + t >= n_step) break;
            const int ch = 32 * (s0 + t) + 8 * ln.q;
            GOp<OPG> pp[NB], pm[NB];
            if constexpr (GATED) {
                const v4f a0 = *reinterpret_cast<const v4f*>(gc + (int64_t)anchor * row_stride + ch);
                const v4f a1 = *reinterpret_cast<const v4f*>(gc + (int64_t)anchor * row_stride + ch + 4);
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    const int64_t off = (int64_t)rowc[i] * row_stride + ch;
                    const v4f g0 = *reinterpret_cast<const v4f*>(gc + off);
                    const v4f g1 = *reinterpret_cast<const v4f*>(gc + off + 4);
                    float kv[8], up[8], dn[8];
                    widen_key8<K16>(raw[t][i], is_f16, kv);
#pragma unroll
                    for (int r = 0; r < 8; ++r) {
                        const float d = ((r < 4) ? (g0[r] - a0[r]) : (g1[r - 4] - a1[r - 4])) * LOG2E;
                        const float kk = kv[r] * keep[i];
                        up[r] = kk * __builtin_amdgcn_exp2f(d);
                        dn[r] = kk * __builtin_amdgcn_exp2f(-d);
                    }
                    pp[i] = gpack<OPG>(up);
                    pm[i] = gpack<OPG>(dn);
                }
            } else {
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    float kv[8];
                    widen_key8<K16>(raw[t][i], is_f16, kv);
#pragma unroll
                    for (int r = 0; r < 8; ++r) kv[r] *= keep[i];
                    pp[i] = gpack<OPG>(kv);  // exact: OPG is the keys' own type
                    pm[i] = pp[i];
                }
            }
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int j = 0; j <= i; ++j) {
                    if (need_tile<NB, METHOD>(i, j, false)) out.n[tix(i, j)] = gstep<OPG>(pp[i], pm[j], out.n[tix(i, j)]);
                    if (need_tile<NB, METHOD>(i, j, true)) out.t[tix(i, j)] = gstep<OPG>(pm[j], pp[i], out.t[tix(i, j)]);
                }
        }
    }
}

// With few matrices the four wavefronts of a workgroup form one matrix together.  What is spread over them: the channels, where the
// operands of the products are made (exponentials), each wavefront one k-step (32 channels) of a round, if there are that many; and the products (fp32 matrix
// instructions, beside which nothing else runs), each wavefront some of the tiles, over all channels.  Between the two the operands go
// through LDS.  Every tile's products are added in one chain in the order of the channels, with the same operands as in the
// loops of one wavefront: a matrix's bits do not depend on how many others its call has.
// Bound by what follows on one wavefront, but for the recursions at C = 64, which the four carry on together (team64.hpp), and by these products where they
// are fp32.  With a recursion on one wavefront, 256 matrices of C = 64, d_k = 128, one
// wavefront / four: per-channel gate 10.8 / 8.2 us, with fp32 operands 19.2 / 12.7, applied to two right-hand sides 14.6 / 12.0, forward
// substitution 17.9 / 12.1; d_k = 256 without a gate, fp32 keys and operands 22.4 / 11.8, bf16 8.1 / 6.8.  512 matrices: 12.1 / 10.2, 20.3 / 16.4,
// 17.5 / 15.4, 19.4 / 15.2, 24.6 / 15.7, 9.2 / 7.7.  (Each wavefront all the products of its own channels and the first adding the sums, another
// order: 8.6, 12.5, 12.3, -, 12.9, 7.4; 11.2, 16.5, 15.8, -, 16.3, 8.5.)
struct Team {
    int w;      // this wavefront of the TEAM_WAVES
    char* lds;  // team_lds_bytes()
};
// The products a method asks for: tile (i, j) in N or T orientation.  Without a gate both operands are the keys, and a diagonal tile is its
// own transpose: one product serves both.
template <int NB, int METHOD, bool GATED> struct GramProducts {
    static constexpr int count_()
    {
        int n = 0;
        for (int i = 0; i < NB; ++i)
            for (int j = 0; j <= i; ++j) n += !GATED && i == j ? 1 : (need_tile<NB, METHOD>(i, j, false) ? 1 : 0) + (need_tile<NB, METHOD>(i, j, true) ? 1 : 0);
        return n;
    }
    static constexpr int COUNT = count_();
    int code[COUNT] = {};  // i | tix(i, j) << 8 | T orientation << 16 | j << 24
    // the product of tile (i, j) in this orientation
    static constexpr int find(int i, int j, bool tr)
    {
        int n = 0;
        for (int a = 0; a < NB; ++a)
            for (int b = 0; b <= a; ++b)
                for (int t = 0; t < 2; ++t) {
                    if (!(!GATED && a == b ? t == 0 : need_tile<NB, METHOD>(a, b, t == 1))) continue;
                    if (a == i && b == j && (t == (tr ? 1 : 0) || (!GATED && a == b))) return n;
                    ++n;
                }
        return -1;
    }
    constexpr GramProducts()
    {
        int n = 0;
        for (int i = 0; i < NB; ++i)
            for (int j = 0; j <= i; ++j)
                for (int tr = 0; tr < 2; ++tr)
                    if (!GATED && i == j ? tr == 0 : need_tile<NB, METHOD>(i, j, tr == 1)) code[n++] = i | (i * (i + 1) / 2 + j) << 8 | j << 24 | tr << 16;
    }
};
// A k-step's operands in LDS, 16 bytes of a lane to a plane of 64 lanes.  Left: NB of them.  Right: without a gate the same.  With a gate, 16-bit
// operands: one per tile; fp32: the factor that depends on the row, one per tile row, the other one (channels only) in the table.
template <int OPG, int NB, bool GATED> struct TeamLds {
    static constexpr int PLANE = 1024, PLANES = OPG == OP_F32 ? 2 : 1, PAIRS = NB * (NB - 1) / 2;
    static constexpr int RIGHT = NB * PLANES * PLANE;
    static constexpr int TABLE = RIGHT + (GATED ? (OPG == OP_F32 ? NB * 2 : NB * (NB + 1) / 2) * PLANE : 0);
    static constexpr int STEP = TABLE + (GATED ? 4 * 8 * (NB + PAIRS) * 4 : 0);
};
// With METHOD's products, of which the finished ones take the operands' place.
template <int OPG, int NB, int METHOD, bool GATED> constexpr int team_lds_bytes()
{
    constexpr int steps = TEAM_WAVES * TeamLds<OPG, NB, GATED>::STEP, tiles = GramProducts<NB, METHOD, GATED>::COUNT * TeamLds<OPG, NB, GATED>::PLANE;
    return steps > tiles ? steps : tiles;
}
template <int OPG> __device__ __forceinline__ void team_write(char* p, const GOp<OPG>& o)
{
    if constexpr (OPG == OP_F32) {  // two planes
        *reinterpret_cast<v4f*>(p) = v4f{o.x[0], o.x[1], o.x[2], o.x[3]};
        *reinterpret_cast<v4f*>(p + 1024) = v4f{o.x[4], o.x[5], o.x[6], o.x[7]};
    } else {
        *reinterpret_cast<decltype(o.x)*>(p) = o.x;
    }
}
template <int OPG> __device__ __forceinline__ GOp<OPG> team_read(const char* p)
{
    if constexpr (OPG == OP_F32) {
        const v4f a = *reinterpret_cast<const v4f*>(p), b = *reinterpret_cast<const v4f*>(p + 1024);
        return GOp<OPG>{{a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]}};
    } else {
        GOp<OPG> o;
        o.x = *reinterpret_cast<const decltype(o.x)*>(p);
        return o;
    }
}

// P products per wavefront over STEPS k-steps, a group's operands on their way while the group before is multiplied.
template <int OPG, int NB, bool GATED, int P, int STEPS> __device__ __forceinline__ void team_products(v4f (&acc)[P], const int (&code)[P], const char* lds, Lane ln)
{
    typedef TeamLds<OPG, NB, GATED> LY;
    constexpr bool FACTORS = GATED && OPG == OP_F32;
    constexpr int GROUP = OPG == OP_F32 ? 1 : 4, PER_STEP = (P + GROUP - 1) / GROUP;
    const int lane = 16 * (16 * ln.q + ln.n);
    GOp<OPG> left[2][GROUP], right[2][GROUP];
    v4f factor[2][GROUP][2];
    const auto fetch = [&](int k) {
        const char* const at = lds + k / PER_STEP * LY::STEP;
#pragma unroll
        for (int g = 0; g < GROUP; ++g) {
            const int p = k % PER_STEP * GROUP + g;
            if (p >= P) break;
            const int i = code[p] & 0xff, j = code[p] >> 24, tile = (code[p] >> 8) & 0xff;
            const bool tr = !FACTORS && ((code[p] >> 16) & 1);  // (here by exchanging the addresses)
            const int a = i * LY::PLANES * LY::PLANE, b = !GATED ? j * LY::PLANES * LY::PLANE : LY::RIGHT + (FACTORS ? j * LY::PLANES : tile) * LY::PLANE;
            left[k & 1][g] = team_read<OPG>(at + (tr ? b : a) + lane);
            right[k & 1][g] = team_read<OPG>(at + (tr ? a : b) + lane);
            if constexpr (FACTORS) {  // (a diagonal tile's is 1: what is read in its place is an anchor)
                const float* const f = reinterpret_cast<const float*>(at + LY::TABLE) + ln.q * 8 * (NB + LY::PAIRS) + 8 * (i == j ? 0 : NB + tile - i);
                factor[k & 1][g][0] = *reinterpret_cast<const v4f*>(f);
                factor[k & 1][g][1] = *reinterpret_cast<const v4f*>(f + 4);
            }
        }
    };
    fetch(0);
#pragma unroll
    for (int k = 0; k < STEPS * PER_STEP; ++k) {
        if (k + 1 < STEPS * PER_STEP) fetch(k + 1);
#pragma unroll
        for (int g = 0; g < GROUP; ++g) {
            const int p = k % PER_STEP * GROUP + g;
            if (p >= P) break;
            GOp<OPG>&a = left[k & 1][g], &b = right[k & 1][g];
            if constexpr (FACTORS) {
                if ((code[p] & 0xff) != code[p] >> 24) {
#pragma unroll
                    for (int r = 0; r < 8; ++r) b.x[r] *= factor[k & 1][g][r / 4][r % 4];
                }
                acc[p] = (code[p] >> 16) & 1 ? gstep<OPG>(b, a, acc[p]) : gstep<OPG>(a, b, acc[p]);
            } else {
                acc[p] = gstep<OPG>(a, b, acc[p]);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// The products of one matrix by the team, left in LDS in the order of GramProducts (team_product).  Every wavefront of the workgroup comes here, with the
// same matrix: the barriers are the workgroup's, the last one behind the products.
// HALF_ROWS: a lane's eight channels of a k-step are 4q .. 4q + 3 and 16 + 4q .. 16 + 4q + 3, not 8q .. 8q + 7 (the order of the products of the kernels
// that keep fp32 keys in registers).
template <int OPG, int NB, int METHOD, bool K16, bool GATED, bool HALF_ROWS = false>
__device__ __forceinline__ void team_gram_products(const void* Kc, bool is_f16, const float* gc, int64_t row_stride, int n_step, Lane ln, int valid,
                                                   const Team& team)
{
    typedef TeamLds<OPG, NB, GATED> LY;
    constexpr float LOG2E = 1.44269504088896340736f;
    static constexpr GramProducts<NB, METHOD, GATED> list;
    constexpr int COUNT = list.COUNT, SIZE = TEAM_WAVES, P = (COUNT + SIZE - 1) / SIZE;  // products in all, at most per wavefront
    const int lane = 16 * (16 * ln.q + ln.n);
    char* const mine = team.lds + team.w * LY::STEP;
    int rowc[NB];
    float keep[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int row = 16 * i + ln.n;
        rowc[i] = row < valid ? row : valid - 1;
        keep[i] = row < valid ? 1.f : 0.f;
    }
    RawKey8<K16> raw[NB];
    v4f G[NB][2];
    const auto load = [&](int s) {
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int64_t off = (int64_t)rowc[i] * row_stride + 32 * s;
            if constexpr (HALF_ROWS) {
                raw[i].a = *reinterpret_cast<const v4f*>(static_cast<const float*>(Kc) + off + 4 * ln.q);
                raw[i].b = *reinterpret_cast<const v4f*>(static_cast<const float*>(Kc) + off + 16 + 4 * ln.q);
            } else {
                raw[i] = load_key8<K16>(Kc, off + 8 * ln.q);
            }
            if constexpr (GATED) {
                G[i][0] = *reinterpret_cast<const v4f*>(gc + off + 8 * ln.q);
                G[i][1] = *reinterpret_cast<const v4f*>(gc + off + 8 * ln.q + 4);
            }
        }
    };
    const auto operands = [&]() {
        if constexpr (!GATED) {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                float kv[8];
                widen_key8<K16>(raw[i], is_f16, kv);
#pragma unroll
                for (int r = 0; r < 8; ++r) kv[r] = !HALF_ROWS ? kv[r] * keep[i] : 16 * i + ln.n < valid ? kv[r] : 0.f;
                team_write<OPG>(mine + i * LY::PLANES * LY::PLANE + lane, gpack<OPG>(kv));
            }
        } else {  // (as in accumulate_gated_gram64)
            constexpr int NE = 8 * LY::PAIRS;
            float* const anc = reinterpret_cast<float*>(mine + LY::TABLE) + ln.q * (8 * NB + NE);
            float* const fac = anc + 8 * NB;
            if (ln.n == 0) {
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    *reinterpret_cast<v4f*>(&anc[8 * i]) = G[i][0];
                    *reinterpret_cast<v4f*>(&anc[8 * i + 4]) = G[i][1];
                }
            }
            wave_lds_sync();
#pragma unroll
            for (int k = 0; k < (NE + 15) / 16; ++k) {
                const int e = ln.n + 16 * k, p = e >> 3, r = e & 7;
                if (e < NE) {
                    const int hi = p >= 3 ? 3 : (p >= 1 ? 2 : 1), lo = p - hi * (hi - 1) / 2;
                    fac[e] = __builtin_amdgcn_exp2f((anc[8 * hi + r] - anc[8 * lo + r]) * LOG2E);
                }
            }
            wave_lds_sync();
            float v[NB][8];
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                float kv[8], u[8];
                widen_key8<K16>(raw[i], is_f16, kv);
                const v4f a0 = *reinterpret_cast<const v4f*>(&anc[8 * i]), a1 = *reinterpret_cast<const v4f*>(&anc[8 * i + 4]);
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    const float kk = kv[r] * keep[i];
                    const float e = (G[i][r / 4][r % 4] - (r < 4 ? a0[r] : a1[r - 4])) * LOG2E;
                    u[r] = kk * __builtin_amdgcn_exp2f(e);
                    v[i][r] = kk * __builtin_amdgcn_exp2f(-e);
                }
                team_write<OPG>(mine + i * LY::PLANES * LY::PLANE + lane, gpack<OPG>(u));
                if constexpr (OPG == OP_F32) team_write<OPG>(mine + LY::RIGHT + i * LY::PLANES * LY::PLANE + lane, gpack<OPG>(v[i]));
            }
            if constexpr (OPG != OP_F32) {
#pragma unroll
                for (int i = 0; i < NB; ++i)
#pragma unroll
                    for (int j = 0; j <= i; ++j) {
                        float dn[8];
                        if (i == j) {
#pragma unroll
                            for (int r = 0; r < 8; ++r) dn[r] = v[j][r];
                        } else {
                            const int p = i * (i - 1) / 2 + j;
                            const v4f f0 = *reinterpret_cast<const v4f*>(&fac[8 * p]), f1 = *reinterpret_cast<const v4f*>(&fac[8 * p + 4]);
#pragma unroll
                            for (int r = 0; r < 8; ++r) dn[r] = v[j][r] * (r < 4 ? f0[r] : f1[r - 4]);
                        }
                        team_write<OPG>(mine + LY::RIGHT + tix(i, j) * LY::PLANE + lane, gpack<OPG>(dn));
                    }
            }
        }
    };

    const int first = team.w * COUNT / SIZE, end = (team.w + 1) * COUNT / SIZE;
    int code[P];
    v4f acc[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {  // (a wavefront with a product fewer does its last one twice)
        const int k = first + p < end ? first + p : first < end ? end - 1 : 0;
        code[p] = list.code[k];
        acc[p] = zero4();
    }
    if (team.w < n_step) load(team.w);
#pragma unroll 1
    for (int s0 = 0; s0 < n_step; s0 += SIZE) {
        const int s = s0 + team.w, steps = n_step - s0;
        if (s < n_step) operands();
        if (s + SIZE < n_step) load(s + SIZE);
        __syncthreads();
        if (steps >= SIZE) {
            team_products<OPG, NB, GATED, P, SIZE>(acc, code, team.lds, ln);
        } else {
            if (steps >= 2) team_products<OPG, NB, GATED, P, 2>(acc, code, team.lds, ln);
            if (steps & 1) team_products<OPG, NB, GATED, P, 1>(acc, code, team.lds + (steps - 1) * LY::STEP, ln);
        }
        __syncthreads();  // the operands have been read
    }
#pragma unroll
    for (int p = 0; p < P; ++p)
        if (first + p < end) *reinterpret_cast<v4f*>(team.lds + (first + p) * LY::PLANE + lane) = acc[p];
    __syncthreads();
}

// Product k of those.
template <int OPG, int NB, bool GATED> __device__ __forceinline__ v4f team_product(const Team& team, int k, Lane ln)
{
    return *reinterpret_cast<const v4f*>(team.lds + k * TeamLds<OPG, NB, GATED>::PLANE + 16 * (16 * ln.q + ln.n));
}

// All tiles, complete on the team's first wavefront; false for the others, which are done.
template <int OPG, int NB, int METHOD, bool K16, bool GATED, bool HALF_ROWS = false>
__device__ __forceinline__ bool team_gram(PreA<NB>& out, const void* Kc, bool is_f16, const float* gc, int64_t row_stride, int n_step, Lane ln, int valid,
                                          const Team& team)
{
    team_gram_products<OPG, NB, METHOD, K16, GATED, HALF_ROWS>(Kc, is_f16, gc, row_stride, n_step, ln, valid, team);
    if (team.w > 0) return false;
    int n = 0;
    const auto next = [&]() { return team_product<OPG, NB, GATED>(team, n++, ln); };
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j <= i; ++j) {
            if (!GATED && i == j) {
                out.n[tix(i, j)] = out.t[tix(i, j)] = next();
                continue;
            }
            if (need_tile<NB, METHOD>(i, j, false)) out.n[tix(i, j)] = next();
            if (need_tile<NB, METHOD>(i, j, true)) out.t[tix(i, j)] = next();
        }
    wave_lds_sync();
    return true;
}
// TEAM: formed by the workgroup's wavefronts together; false for those that are done.
template <int OPG, int NB, int METHOD, bool TEAM>
__device__ __forceinline__ bool build_A_per_channel(PreA<NB>& out, const void* Kc, int kd, const float* gc, int64_t row_stride,
                                                    const float* bc, int64_t tok_stride, int d_k, float* lds, Lane ln, int valid, bool ahead, const Team& team)
{
    constexpr int C = 16 * NB;
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j <= i; ++j) {
            out.n[tix(i, j)] = zero4();
            out.t[tix(i, j)] = zero4();
        }
    if constexpr (TEAM) {
        if (!(kd == OP_F32 ? team_gram<OPG, NB, METHOD, false, true>(out, Kc, false, gc, row_stride, d_k / 32, ln, valid, team)
                           : team_gram<OPG, NB, METHOD, true, true>(out, Kc, kd == OP_F16, gc, row_stride, d_k / 32, ln, valid, team)))
            return false;
    } else if (kd == OP_F32) {
        accumulate_gated_gram<OPG, NB, METHOD, false>(out, Kc, false, gc, row_stride, d_k / 32, ln, valid, lds, ahead);
    } else {
        accumulate_gated_gram<OPG, NB, METHOD, true>(out, Kc, kd == OP_F16, gc, row_stride, d_k / 32, ln, valid, lds, ahead);
    }
    // beta_i row scaling and the strictly-lower mask
    const int l = 16 * ln.q + ln.n;
#pragma unroll
    for (int t = l; t < C; t += 64) lds[t] = t < valid ? bc[t * tok_stride] : 0.f;
    wave_lds_sync();
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const float bn = lds[16 * i + ln.n];
        const v4f bq = *reinterpret_cast<const v4f*>(&lds[16 * i + 4 * ln.q]);
#pragma unroll
        for (int j = 0; j <= i; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const bool lowN = (i != j) || (4 * ln.q + r > ln.n), lowT = (i != j) || (ln.n > 4 * ln.q + r);
                out.n[tix(i, j)][r] = lowN ? bq[r] * out.n[tix(i, j)][r] : 0.f;
                out.t[tix(i, j)][r] = lowT ? bn * out.t[tix(i, j)][r] : 0.f;
            }
    }
    wave_lds_sync();
    return true;
}

// Scalar / no-gate kinds for any d_k (multiple of 32): Gram tiles accumulated 32 channels at a time
// in a run-time loop with the stored keys as operands, then the scalar gate.  KD = type of K.
template <int KD, int NB, int METHOD, bool TEAM>
__device__ __forceinline__ bool build_A_scalar_any_dk(PreA<NB>& out, const void* Kc, int64_t row_stride, const float* bc,
                                                      const float* gc, int64_t tok_stride, int d_k, float* lds, Lane ln, int valid, const Team& team)
{
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j <= i; ++j) {
            out.n[tix(i, j)] = zero4();
            out.t[tix(i, j)] = zero4();
        }
    if constexpr (!TEAM) {
        accumulate_gated_gram<KD, NB, METHOD, KD != OP_F32, false>(out, Kc, KD == OP_F16, nullptr, row_stride, d_k / 32, ln, valid);
    } else {
        bool more = true;
        if (KD == OP_F32 && NB == 4 && d_k == FP32_KEYS_TEAM_DK) {  // in the order of the kernel that these keys have at this size
            if constexpr (KD == OP_F32 && NB == 4) more = team_gram<KD, NB, METHOD, false, false, true>(out, Kc, false, nullptr, row_stride, d_k / 32, ln, valid, team);
        } else {
            more = team_gram<KD, NB, METHOD, KD != OP_F32, false>(out, Kc, KD == OP_F16, nullptr, row_stride, d_k / 32, ln, valid, team);
        }
        if (!more) return false;
    }
    GateVec<NB> gate;
    gate.load(bc, gc, tok_stride, lds, ln, valid);
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j <= i; ++j) {
            if (need_tile<NB, METHOD>(i, j, false)) out.n[tix(i, j)] = gate.template apply<false>(i, j, out.n[tix(i, j)], ln);
            if (need_tile<NB, METHOD>(i, j, true)) out.t[tix(i, j)] = gate.template apply<true>(i, j, out.t[tix(i, j)], ln);
        }
    return true;
}

// ---------------------------------------------------------------------------------------------
// Result store.  Tm: first element of this matrix's T.  The register tiles (N or T orientation,
// IS_T(i, j)) of one 16-row strip are transposed through a wave-private LDS patch into plain
// rows, and the strip leaves as four 1 KB-contiguous streaming stores (16 B per lane): whole
// cache lines written by one instruction stream to HBM markedly faster than the 64-byte pieces
// a tile-shaped store produces.  Diagonal tiles get an exact unit diagonal and exact zeros above
// it; columns right of the diagonal tile are zero-filled.
// lds: store_lds_floats<NB>() floats.
// ---------------------------------------------------------------------------------------------
// Streaming stores of the result.  Whole 16-byte pieces of full rows go out non-temporal and at
// system scope (written through the caches: T is consumed by a later kernel, never re-read here);
// measured with a same-pattern data mover ~4 % faster than the non-temporal hint alone and ~11 %
// faster than plain stores.  They are raw buffer stores over a descriptor that spans exactly this
// matrix (the cache-policy bits are an argument of the builtin, and the compiler, which sees the
// instruction, keeps the wait states a wide store needs before its data registers are rewritten;
// offsets outside the matrix would be dropped by the hardware's range check).  The 4-byte stores of
// whole rows one by one (forward substitution at C = 16 and its shuffle form) keep the plain non-temporal hint (partial lines written
// through measured slower).
constexpr int CACHE_SC0_SC1_NT = 1 | 2 | 16;  // gfx950 buffer-instruction cache-policy bits: sc0, nt, sc1

// One output matrix: its first byte and its element type (OP_F32, or OP_F16 / OP_BF16 when the caller
// asked for a 16-bit result: the fp32 values are rounded to nearest even on the way out).
struct Out {
    void* base;
    int dt;
};
__device__ __forceinline__ Out out_matrix(float* T, int64_t m, int C, int out_dt)
{
    return Out{reinterpret_cast<char*>(T) + m * C * C * (out_dt == OP_F32 ? 4 : 2), out_dt};
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t matrix_buffer(Out Tm, int C)
{
    return __builtin_amdgcn_make_buffer_rsrc(Tm.base, 0, C * C * (Tm.dt == OP_F32 ? 4 : 2), 0x00020000);  // raw buffer
}
// byte offset = lane_offset (the same for every store of a strip) + uniform_offset (a constant of the strip and row group).
// Both go into the vector offset, the instruction's scalar offset stays the immediate zero.  A 16-byte store whose scalar
// offset is a register is not safe here: the compiler places no wait state between such a store and a vector-ALU write
// of its data registers (it guards only the immediate form), and with a write in the very next slot the store now and
// then sent the new value of its first data register: about one matrix in 10^6 came out with the next strip's values
// in 16 of its elements.  With the immediate form the compiler inserts the wait state itself.  (The scalar form followed by
// an explicit two-slot wait that keeps the data registers alive measured the same: +0.9 % at C = 64, -0.9 % at C = 128.)
__device__ __forceinline__ void stream_store(v4u v, __amdgpu_buffer_rsrc_t out, int lane_offset, int uniform_offset = 0)
{
    __builtin_amdgcn_raw_buffer_store_b128(v, out, lane_offset + uniform_offset, 0, CACHE_SC0_SC1_NT);
}
__device__ __forceinline__ void stream_store(v4f v, __amdgpu_buffer_rsrc_t out, int lane_offset, int uniform_offset = 0)
{
    stream_store(__builtin_bit_cast(v4u, v), out, lane_offset, uniform_offset);
}
__device__ __forceinline__ void stream_store(float v, float* p) { __builtin_nontemporal_store(v, p); }
// Row stride of the patch in floats.  C <= 32 has a patch of its own size: with one that fits C = 128 its wavefronts would clear
// 8 KB of LDS for a 1 or 4 KB result, and 18 of them would fill a compute unit (65536 matrices of C = 16, forward
// substitution: 41.9 us).  C = 64 keeps the larger one: it holds four wavefronts' workgroups to four per
// compute unit, and those kernels run slower with more (see occupancy_pad_bytes).
template <int NB> __host__ __device__ constexpr int store_ld() { return NB <= 2 ? 16 * NB + 4 : 16 * 8 + 4; }
template <int NB> __host__ __device__ constexpr int store_lds_floats() { return 16 * store_ld<NB>(); }
constexpr int STORE_LDS_FLOATS = store_lds_floats<8>();

// Zero the strip patch.  Strips stored afterwards in ascending order then find zeros right of their diagonal tile (strip
// i only writes tiles 0..i), which spares them a select per stored element.
template <int NB> __device__ __forceinline__ void zero_strip_patch(float* lds, Lane ln)
{
    constexpr int VECS = store_lds_floats<NB>() / 4;
    const int lane = 16 * ln.q + ln.n;
#pragma unroll
    for (int k = 0; k < (VECS + 63) / 64; ++k) {
        const int p = 64 * k + lane;
        if (p < VECS) *reinterpret_cast<v4f*>(&lds[4 * p]) = zero4();
    }
    wave_lds_sync();
}

// Strip i, which lies in the patch as 16 plain rows, to memory.  ZEROED: the patch holds zeros right of tile i.
template <int NB, bool ZEROED, int LD = store_ld<NB>()> __device__ __forceinline__ void flush_strip(Out Tm, int i, const float* lds, Lane ln)
{
    constexpr int C = 16 * NB;
    const int lane = 16 * ln.q + ln.n;
    const __amdgpu_buffer_rsrc_t out = matrix_buffer(Tm, C);
    wave_lds_sync();
    if (Tm.dt == OP_F32) {
        // rows 16i .. 16i+15, C floats each: C/4 lanes per row, 256/C rows per instruction
        constexpr int LPR = C / 4, RPI = 64 / LPR;
#pragma unroll
        for (int k = 0; k < 16 / RPI; ++k) {
            const int rr = RPI * k + lane / LPR, cc = 4 * (lane % LPR);
            // unconditional read (columns right of the diagonal tile hold stale patch contents), then a select
            v4f v = *reinterpret_cast<const v4f*>(&lds[rr * LD + cc]);
            if (!ZEROED && cc >= 16 * (i + 1)) v = zero4();
            stream_store(v, out, ((lane / LPR) * C + cc) * 4, (16 * i + RPI * k) * C * 4);
        }
    } else {
        // 16-bit result: 8 elements (16 bytes) per lane, C/8 lanes per row
        constexpr int LPR = C / 8, RPI = 64 / LPR, ITER = RPI >= 16 ? 1 : 16 / RPI;
#pragma unroll
        for (int k = 0; k < ITER; ++k) {
            const int rr = RPI * k + lane / LPR, cc = 8 * (lane % LPR);
            if (RPI > 16 && rr >= 16) continue;  // C = 16: more lanes than the strip has 16-byte pieces
            v4f a = *reinterpret_cast<const v4f*>(&lds[rr * LD + cc]);
            v4f b = *reinterpret_cast<const v4f*>(&lds[rr * LD + cc + 4]);
            if (!ZEROED && cc >= 16 * (i + 1)) a = zero4();
            if (!ZEROED && cc + 4 >= 16 * (i + 1)) b = zero4();
            const v4u p = Tm.dt == OP_F16 ? v4u{pack2_f16(a[0], a[1]), pack2_f16(a[2], a[3]), pack2_f16(b[0], b[1]), pack2_f16(b[2], b[3])}
                                          : v4u{pack2_bf16(a[0], a[1]), pack2_bf16(a[2], a[3]), pack2_bf16(b[0], b[1]), pack2_bf16(b[2], b[3])};
            stream_store(p, out, ((lane / LPR) * C + cc) * 2, (16 * i + RPI * k) * C * 2);
        }
    }
    wave_lds_sync();
}

// Tile (i, j) of strip i into the patch, in T orientation or not; a diagonal tile gets ones on its diagonal and zeros above.  For the kernels that
// spread a matrix over wavefronts.  store_strip does the same in its own words: by way of this function the standalone Neumann product with
// 16-bit operands takes 131 registers in place of 128 and loses a wavefront per SIMD (C = 64, 8192 fp32 matrices 33.3 -> 35.2 us).
template <int LD> __device__ __forceinline__ void strip_tile(float* lds, int i, int j, v4f v, bool is_t, Lane ln)
{
    if (is_t) {  // v[r] = T[16i + n][16j + 4q + r]
        if (i == j) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int rr = ln.n, cc = 4 * ln.q + r;
                v[r] = (rr == cc) ? 1.f : ((rr > cc) ? v[r] : 0.f);
            }
        }
        *reinterpret_cast<v4f*>(&lds[ln.n * LD + 16 * j + 4 * ln.q]) = v;
    } else {     // v[r] = T[16i + 4q + r][16j + n]
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int rr = 4 * ln.q + r, cc = ln.n;
            float x = v[r];
            if (i == j) x = (rr == cc) ? 1.f : ((rr > cc) ? x : 0.f);
            lds[rr * LD + 16 * j + cc] = x;
        }
    }
}

// One strip: tiles (i, 0..i) in row[0..i], tile j in T orientation when row_is_t(j).
// ZEROED: the patch holds zeros right of tile i (zero_strip_patch, then strips in ascending order).
template <int NB, bool ZEROED = false, class RowIsT>
__device__ __forceinline__ void store_strip(Out Tm, int i, const v4f (&row)[NB], RowIsT row_is_t, float* lds, Lane ln,
                                            float diag = 1.f)
{
    constexpr int LD = store_ld<NB>();
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        if (j > i) break;
        v4f v = row[j];
        if (row_is_t(j)) {  // v[r] = T[16i + n][16j + 4q + r]
            if (i == j) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int rr = ln.n, cc = 4 * ln.q + r;
                    v[r] = (rr == cc) ? diag : ((rr > cc) ? v[r] : 0.f);
                }
            }
            *reinterpret_cast<v4f*>(&lds[ln.n * LD + 16 * j + 4 * ln.q]) = v;
        } else {            // v[r] = T[16i + 4q + r][16j + n]
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int rr = 4 * ln.q + r, cc = ln.n;
                float x = v[r];
                if (i == j) x = (rr == cc) ? diag : ((rr > cc) ? x : 0.f);
                lds[rr * LD + 16 * j + cc] = x;
            }
        }
    }
    flush_strip<NB, ZEROED>(Tm, i, lds, ln);
}

template <int NB, class IsT>
__device__ __forceinline__ void store_result(Out Tm, const v4f (&Tt)[NB * (NB + 1) / 2], IsT is_t, float* lds, Lane ln,
                                             float diag = 1.f)
{
    if constexpr (NB == 1) {
        // a single tile in T orientation is already 16 rows of four 16-byte pieces: no turn through LDS (C = 16, 65536 matrices,
        // fp32 operands, standalone blocked recursion 29 -> 21 us together with the smaller patch)
        if (is_t(0, 0)) {
            const __amdgpu_buffer_rsrc_t out = matrix_buffer(Tm, 16);
            v4f v;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int cc = 4 * ln.q + r;
                v[r] = (ln.n == cc) ? diag : ((ln.n > cc) ? Tt[0][r] : 0.f);
            }
            const int e = ln.n * 16 + 4 * ln.q;
            if (Tm.dt == OP_F32)
                stream_store(v, out, e * 4);
            else
                __builtin_amdgcn_raw_buffer_store_b64(Tm.dt == OP_F16 ? v2u{pack2_f16(v[0], v[1]), pack2_f16(v[2], v[3])}
                                                                      : v2u{pack2_bf16(v[0], v[1]), pack2_bf16(v[2], v[3])},
                                                      out, e * 2, 0, CACHE_SC0_SC1_NT);
            return;
        }
    }
    zero_strip_patch<NB>(lds, ln);
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        v4f row[NB];
#pragma unroll
        for (int j = 0; j <= i; ++j) row[j] = Tt[tix(i, j)];
        store_strip<NB, true>(Tm, i, row, [&](int j) { return is_t(i, j); }, lds, ln, diag);
    }
}

// ---------------------------------------------------------------------------------------------
// Forward substitution in fp32, 16 rows at a time: for tile row i, the products with the rows above it,
//   S_ik = A_ik T_kk + ... + A_i,i-1 T_i-1,k   (k < i; S_ii = 0),
// in fp32 matrix-core instructions, then (I + A_ii) T_ik = -S_ik (T_ii: = I) row by row in vector arithmetic, lane group p
// solving tile 4 g + p of the row and lane n its column n.  A row of A is needed only for its own row of T, so T takes A's place in
// registers.
//
// The order of the sums is what makes it as accurate as substitution row by row (an fp32 matrix instruction is a chain of four
// multiply-adds, contraction slot 0 first): a tile contributes two sums of 8 terms, each taken from the last row up and started from
// zero, and the sums are added in ascending order of the rows; so are the row's own tile's, last.  Error against 64 bits below the
// diagonal (A given in fp32, C = 128 / 64 / 32, in brackets one chain per element row by row from the first): correlated keys
// without decay 2.27e-7 (2.34e-7) / 1.55e-7 (1.60e-7) / 1.01e-7 (1.03e-7), Gaussian keys 6.8e-8 (1.75e-7) / 4.8e-8 (1.20e-7) /
// 3.6e-8 (8.0e-8).  One chain over all tiles, and the inverse of the diagonal block in place of its solve, take 3.04e-7 / 2.00e-7 /
// 1.19e-7 on the former; that inverse also spreads an infinity or NaN of A over rows above its own, where here only rows that
// depend on it see it.
//
// Bound by memory at C <= 64, at C = 128 by the serial rows of its two wavefronts per SIMD (4519 vector and 480 matrix instructions a
// matrix; vector unit 0.35, matrix cores 0.25 busy).  2048 fused matrices of C = 128: 42.7 us (row by row throughout, 10144
// dependent multiply-adds and 2536 LDS broadcasts a lane, one wavefront per SIMD: 140; with the block's inverse 41.7), on the
// workload of correlated keys, 8192, 192 us (167 with the inverse); a call of 32: 21 us (63, 15); standalone fp32, 8192 matrices
// 179 us (262); C = 64 fused, 16384: 93-100 us (125, 101), standalone 45 us (54, 44; 8192).
// ---------------------------------------------------------------------------------------------

// Four registers against the four lane groups: x[p] of lane group q <- x[q] of lane group p.
__device__ __forceinline__ void turn_groups(float (&x)[4])
{
    const auto u = [&](int r) { return __builtin_bit_cast(uint32_t, x[r]); };
    const auto a = __builtin_amdgcn_permlane32_swap(u(0), u(2), false, false), b = __builtin_amdgcn_permlane32_swap(u(1), u(3), false, false);
    const auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false), d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
    const uint32_t y[4] = {c[0], c[1], d[0], d[1]};
#pragma unroll
    for (int r = 0; r < 4; ++r) x[r] = __builtin_bit_cast(float, (uint32_t)y[r]);
}

template <int NB> constexpr int forward_lds_floats() { return NB == 1 ? 16 * LEAF_LD : store_lds_floats<NB>() + 16 * LEAF_LD; }

// The products A_I+1,j T_jk that do not need tile row I, in the order of their sums.
template <int I> struct ForwardProducts {
    static constexpr int count = I * (I + 1) / 2;
    int k[count + 1] = {}, j[count + 1] = {};
    constexpr ForwardProducts()
    {
        int n = 0;
        for (int kk = 0; kk < I; ++kk)
            for (int jj = kk; jj < I; ++jj, ++n) {
                k[n] = kk;
                j[n] = jj;
            }
    }
};

// The two halves of a tile product (operands: element r of lane group q is row 4 r + 3 - q of the contraction).
__device__ __forceinline__ void forward_product(v4f a, v4f b, v4f& low, v4f& high)
{
    low = __builtin_amdgcn_mfma_f32_16x16x4f32(a[1], b[1], zero4(), 0, 0, 0);
    high = __builtin_amdgcn_mfma_f32_16x16x4f32(a[3], b[3], zero4(), 0, 0, 0);
    low = __builtin_amdgcn_mfma_f32_16x16x4f32(a[0], b[0], low, 0, 0, 0);
    high = __builtin_amdgcn_mfma_f32_16x16x4f32(a[2], b[2], high, 0, 0, 0);
}

// Tile row I.  T: tile rows of T above it as right operands, row I and the rows below it of A, row I's as left operands.  sums: S_Ik but
// for the terms of row I - 1.
template <int NB, int I>
__device__ __forceinline__ void forward_tile_row(v4f (&T)[NB * (NB + 1) / 2], v4f (&sums)[NB], Out Tm, float* patch, float* leaf, Lane ln)
{
    constexpr int LD = store_ld<NB>();
    constexpr int GROUPS = I / 4 + 1;
    const int lane = 16 * ln.q + ln.n;
    *reinterpret_cast<v4f*>(&leaf[ln.n * LEAF_LD + 4 * ln.q]) = T[tix(I, I)];
#pragma unroll
    for (int k = 0; k < I; ++k) {
        if (NB == 8 && k % 2 == 0) __builtin_amdgcn_sched_barrier(0);
        v4f low, high;
        forward_product(T[tix(I, I - 1)], T[tix(I - 1, k)], low, high);
        sums[k] = (k == I - 1 ? low : sums[k] + low) + high;
    }
    if constexpr (I + 1 < NB) {
#pragma unroll
        for (int j = 0; j <= I; ++j) {
            if (NB == 8 && j % 4 == 0) __builtin_amdgcn_sched_barrier(0);
            v4f& a = T[tix(I + 1, j)];
            float x[4] = {a[3], a[2], a[1], a[0]};
            turn_groups(x);
            a = v4f{x[0], x[1], x[2], x[3]};
        }
    }
    float t[GROUPS][16];  // S (the unit matrix for the diagonal tile), then T, of tile 4 g + q: column n, all 16 rows
    Lane col = ln;
    asm volatile("" : "+v"(col.n));  // (what follows from it is not worth registers from one tile row to the next)
    const v4f unit_tile = identity_tile(col);
    int unit[GROUPS];     // the row of the column's diagonal element: -1 left of the diagonal tile, 16 right of it
#pragma unroll
    for (int g = 0; g < GROUPS; ++g) {
        if (NB == 8) __builtin_amdgcn_sched_barrier(0);
        unit[g] = 4 * g + ln.q < I ? -1 : 4 * g + ln.q == I ? col.n : 16;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float x[4];
#pragma unroll
            for (int p = 0; p < 4; ++p) x[p] = 4 * g + p < I ? sums[4 * g + p][r] : 4 * g + p == I ? unit_tile[r] : 0.f;
            turn_groups(x);
#pragma unroll
            for (int p = 0; p < 4; ++p) t[g][4 * p + r] = x[p];
        }
    }
    leaf_lds_sync();
    // The products of the next tile row that do not need this one go between the rows of the solve, so that the matrix cores and
    // the vector unit have work at the same time.  (The fences keep a row's reads of the leaf and its products to that row: all at
    // once they would spill T.)
    static constexpr ForwardProducts<I> list;
    constexpr int count = I + 1 < NB ? list.count : 0;
    static_assert(count <= 32, "at most two products beside a row");
    v4f a[16][4];
    const auto read_row = [&](int row) {
#pragma unroll
        for (int m = 0; m < 4; ++m)
            if (4 * m < row) a[row][m] = *reinterpret_cast<const v4f*>(&leaf[row * LEAF_LD + 4 * m]);
    };
#pragma unroll
    for (int row = 0; row < 16; ++row) {
        __builtin_amdgcn_sched_barrier(0);
        v4f low[2], high[2];
        constexpr int AHEAD = NB < 8 ? 15 : 12;  // rows read a row early: the last ones would not fit at C = 128
        if (row < AHEAD) read_row(row + 1);
        if (row > AHEAD) read_row(row);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int p = row * count / 16 + e;
            if (p < (row + 1) * count / 16) forward_product(T[tix(I + 1, list.j[p])], T[tix(list.j[p], list.k[p])], low[e], high[e]);
        }
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) {
            float below = 0.f, above = 0.f;
#pragma unroll
            for (int m = 7; m >= 0; --m)
                if (m < row) above = __builtin_fmaf(a[row][m / 4][m % 4], t[g][m], above);
#pragma unroll
            for (int m = 15; m >= 8; --m)
                if (m < row) below = __builtin_fmaf(a[row][m / 4][m % 4], t[g][m], below);
            float v = -t[g][row] - (row > 8 ? below + above : above);
            if (4 * g + 3 >= I) {
                asm("" : "+v"(v));  // (a select, no branch around the sums)
                v = unit[g] < row ? v : t[g][row];
            }
            t[g][row] = v;
        }
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int p = row * count / 16 + e;
            if (p < (row + 1) * count / 16) {
                v4f& s = sums[list.k[p]];
                s = (list.j[p] == list.k[p] ? low[e] : s + low[e]) + high[e];
                asm volatile("" : "+v"(s));  // (here: left to the end of the solve, the sums hold their operands' registers until then)
            }
        }
    }
#pragma unroll
    for (int g = 0; g < GROUPS; ++g)
#pragma unroll
        for (int row = 0; row < 16; ++row)
            if (NB >= 4 || lane < 16 * NB) patch[row * LD + 64 * g + lane] = t[g][row];
    flush_strip<NB, true>(Tm, I, patch, ln);
    if constexpr (I + 1 < NB) {
#pragma unroll
        for (int g = 0; g < GROUPS; ++g)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float x[4] = {t[g][4 * r + 3], t[g][4 * r + 2], t[g][4 * r + 1], t[g][4 * r]};
                turn_groups(x);
#pragma unroll
                for (int p = 0; p < 4; ++p)
                    if (4 * g + p <= I) T[tix(I, 4 * g + p)][r] = x[p];
            }
        forward_tile_row<NB, I + 1>(T, sums, Tm, patch, leaf, ln);
    }
}

template <int NB, class ASrc>
__device__ __forceinline__ void forward_substitution(const ASrc& A, Out Tm, float* lds, Lane ln)
{
    if constexpr (NB == 1) {
        // one leaf: its rows are stored as they are finished, without another turn through LDS (a copy per element size: a
        // choice inside the loop splits it into blocks, and all reads of the leaf end up before the first)
        const v4f a = A.template get<true>(0, 0);
        *reinterpret_cast<v4f*>(&lds[ln.n * LEAF_LD + 4 * ln.q]) = a;
        leaf_lds_sync();
        float t[16];
        if (Tm.dt == OP_F32) {
            float* const out = static_cast<float*>(Tm.base) + ln.n;
            solve_leaf_column(lds, ln.n, t, [&](int i) { if (ln.q == 0) __builtin_nontemporal_store(t[i], out + 16 * i); });
        } else {
            uint16_t* const out = static_cast<uint16_t*>(Tm.base) + ln.n;
            solve_leaf_column(lds, ln.n, t, [&](int i) {
                if (ln.q == 0) __builtin_nontemporal_store((uint16_t)(Tm.dt == OP_F16 ? pack2_f16(t[i], 0.f) : pack2_bf16(t[i], 0.f)), out + 16 * i);
            });
        }
    } else {
        // All tiles of A first, from the last tile row up: a source that holds keys needs them ever less then, and A and the
        // remaining keys fit two wavefronts per SIMD at C = 128.
        v4f T[NB * (NB + 1) / 2], sums[NB];
#pragma unroll
        for (int i = NB - 1; i >= 0; --i) {
#pragma unroll
            for (int j = 0; j <= i; ++j) T[tix(i, j)] = A.template get<true>(i, j);
            if (ASrc::kHoldsKeys && NB == 8) __builtin_amdgcn_sched_barrier(0);
        }
        if (NB > 4) zero_strip_patch<NB>(lds, ln);  // (up to four tiles a row, every row writes all of them)
        forward_tile_row<NB, 0>(T, sums, Tm, lds, lds + store_lds_floats<NB>(), ln);
    }
}

// Forward substitution at C = 64 row by row, the row of A broadcast by wavefront shuffles: lane l
// holds A[i][l] of every row i (one coalesced 256-byte load per row, all 63 issued up front) and
// T[:, l]; A[i][j] reaches every lane through a v_readlane of lane j, one shuffle per multiply-add.  Kept as the plain
// shuffle baseline (210 us for 16384 matrices).
__device__ __forceinline__ void forward_substitution_shuffle64(const void* Am, int in_dt, float* Tm, Lane ln)
{
    constexpr int C = 64;
    const int c = 16 * ln.q + ln.n;
    float a[C];  // a[i] = A[i][c] for c < i, else 0
#pragma unroll
    for (int i = 1; i < C; ++i) {
        float v;
        if (in_dt == OP_F32) {
            v = static_cast<const float*>(Am)[i * C + c];
        } else {
            const uint16_t u = static_cast<const uint16_t*>(Am)[i * C + c];
            v = in_dt == OP_F16 ? f16_to_f32(u) : bf16_to_f32(u);
        }
        a[i] = c < i ? v : 0.f;
    }
    float Tc[C];
    Tc[0] = c == 0 ? 1.f : 0.f;
    stream_store(Tc[0], Tm + c);
#pragma unroll
    for (int i = 1; i < C; ++i) {
        float acc = 0.f;
#pragma unroll
        for (int j = 0; j < i; ++j) {
            const float aij = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, a[i]), j));
            acc += aij * Tc[j];
        }
        Tc[i] = (c < i) ? -acc : ((c == i) ? 1.f : 0.f);
        stream_store(Tc[i], Tm + i * C + c);
    }
}

template <int UNUSED = 0>  // a template only so that the header may define it in every translation unit
__global__ __launch_bounds__(64) void k_tri_inv_fwd_shuffle64(const void* __restrict__ A, float* __restrict__ T, int64_t n_mat, int in_dt)
{
    const int64_t m = blockIdx.x;
    if (m >= n_mat) return;
    forward_substitution_shuffle64(static_cast<const char*>(A) + m * 64 * 64 * (in_dt == OP_F32 ? 4 : 2), in_dt, T + m * 64 * 64,
                                   lane_id());
}

// ---------------------------------------------------------------------------------------------
// Kernels
// ---------------------------------------------------------------------------------------------
template <int NB> constexpr int gate_lds_floats() { return 2 * 16 * NB; }

// LDS of one wavefront's inversion: the store patch, which also serves as transpose patch and holds the staged leaves of the
// direct methods (a leaf per tile row, at most four at a time).
template <int NB, int METHOD> constexpr int core_lds_floats()
{
    if (METHOD == M_FWD) return forward_lds_floats<NB>();
    constexpr int leaves = METHOD == M_NEWTON_SCHULZ ? ns_lds_floats<OP_F32, NB>() : (NB < 4 ? NB : 4) * LEAF_STRIDE;
    constexpr int small = leaves > XPOSE_FLOATS ? leaves : XPOSE_FLOATS;
    return store_lds_floats<NB>() > small ? store_lds_floats<NB>() : small;
}

// The team of this wavefront: its workgroup.
__device__ __forceinline__ Team this_team(char* lds) { return Team{__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lds}; }
// (Refined Newton-Schulz with fp32 operands at C = 64 takes more than 256 registers: a compute unit would hold one team of the two.)
template <int OP, int NB, int METHOD, bool REFINE> constexpr bool kda_team() { return NB <= 4 && !(METHOD == M_NEWTON_SCHULZ && NB == 4 && OP == OP_F32 && REFINE); }

// REFINE: one iterative-refinement step after a matrix-product method (C <= 64; at C = 128 a kernel of its own).
template <int OP, int NB, int METHOD, class ASrc, bool REFINE = false>
__device__ __forceinline__ void invert_and_store(const ASrc& src, Out Tm, float* lds, Lane ln, int aux = 0)
{
    constexpr int NT = NB * (NB + 1) / 2;
    if constexpr (METHOD == M_BUILD_A) {
        // the strictly-lower chunk matrix itself (zero diagonal), strip by strip: at most NB tiles alive at a time
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            v4f row[NB];
#pragma unroll
            for (int j = 0; j <= i; ++j) row[j] = src.template get<true>(i, j);
            store_strip<NB>(Tm, i, row, [](int) { return true; }, lds, ln, 0.f);
        }
        return;
    }
    if (METHOD == M_FWD) {
        forward_substitution<NB>(src, Tm, lds, ln);
    } else if (METHOD == M_NEWTON_SCHULZ) {
        v4f Xt[NT];
        newton_schulz<OP, NB>(src, Xt, aux, lds, ln);  // aux = number of iterations
        if constexpr (REFINE) refine_once<OP, NB>(src, Xt, [](int, int) { return false; }, lds, ln);  // (turns every tile)
        store_result<NB>(Tm, Xt, [](int, int) { return REFINE; }, lds, ln);
    } else if (METHOD == M_NEUMANN) {
        v4f Xt[NT];
        neumann<OP, NB>(src, Xt, ln);
        if constexpr (REFINE) refine_once<OP, NB>(src, Xt, [](int, int) { return true; }, lds, ln);
        store_result<NB>(Tm, Xt, [](int, int) { return true; }, lds, ln);
    } else {
        v4f Tt[NT];
        constexpr int LEAF = METHOD == M_MIXED ? LEAF_NEUMANN : METHOD == M_MIXED32 ? LEAF_NEUMANN32 : METHOD == M_BLOCK_DIRECT ? LEAF_FORWARD : LEAF_BLOCK_RECURSIVE;
        // fp32 leaves side by side: four where A is given; two where it comes from keys, so that the first start before the
        // last keys are there; one after the other in the channel-loop kernels at C = 128, which hold all of A beside them
        constexpr int PATCHES = ASrc::kFromMemory ? 4 : ASrc::kHoldsKeys ? 2 : NB == 8 ? 1 : 4;
        static_assert((PATCHES < NB ? PATCHES : NB) * XPOSE_FLOATS <= core_lds_floats<NB, METHOD>(), "a patch per leaf");
        block_recursive<OP, NB, ROOT_T, LEAF, PATCHES>(src, Tt, lds, ln, aux);  // aux = refinement steps on the leaves (mixed recursion)
        if constexpr (REFINE) {
            refine_once<OP, NB>(src, Tt, [](int i, int j) { return result_is_T<NB, ROOT_T>(i, j); }, lds, ln);
            store_result<NB>(Tm, Tt, [](int, int) { return true; }, lds, ln);
        } else {
            store_result<NB>(Tm, Tt, [](int i, int j) { return result_is_T<NB, ROOT_T>(i, j); }, lds, ln);
        }
    }
}

// The matrix-product kernels may be run in place (A and T the same memory: the composed path of the fused entry points),
// so only forward substitution, which never is, declares its two pointers non-aliasing.
template <int METHOD> struct TriInvPointers {
    typedef const void* in;
    typedef float* out;
};
template <> struct TriInvPointers<M_FWD> {
    typedef const void* __restrict__ in;
    typedef float* __restrict__ out;
};

// Wavefronts per SIMD the register allocator has to leave room for.  Newton-Schulz with fp32 operands at C = 64 needs two:
// its matrix-core and its vector instructions take about the same time and overlap only between wavefronts (with the refinement step it
// does not fit).  So does forward substitution at C = 128 (255 registers this way; with the per-channel gate it holds A beside the
// running keys and factors and would spill), and the per-channel kernels at C = 64, whose loads a step ahead take some methods just
// beyond 256.
template <int OP, int NB, int METHOD, bool REFINE, bool PER_CHANNEL = false> constexpr int min_waves_per_simd()
{
    constexpr bool split = METHOD == M_NEWTON_SCHULZ && OP == OP_F32;
    if (NB == 4) return (split || PER_CHANNEL) && !(split && REFINE) ? 2 : 1;
    return METHOD == M_FWD && NB == 8 && !PER_CHANNEL ? 2 : 1;
}

template <int IN, int OP, int NB, int METHOD, bool REFINE = false>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(min_waves_per_simd<OP, NB, METHOD, REFINE>()))) void k_tri_inv(
    typename TriInvPointers<METHOD>::in A, typename TriInvPointers<METHOD>::out T, int64_t n_mat, int in_dt, int aux, int out_dt)
{
    constexpr int C = 16 * NB;
    __shared__ __attribute__((aligned(16))) float lds[core_lds_floats<NB, METHOD>()];
    const int64_t m = blockIdx.x;
    if (m >= n_mat) return;
    const Lane ln = lane_id();
    const void* const base = static_cast<const char*>(A) + m * C * C * (IN == OP_F32 ? 4 : 2);
    const Out Tm = out_matrix(T, m, C, out_dt);
    if constexpr (IN != OP_F32) {
        LoadedA16<IN, OP, NB> src;
        src.load(base, ln);
        invert_and_store<OP, NB, METHOD, LoadedA16<IN, OP, NB>, REFINE>(src, Tm, lds, ln, aux);
    } else if constexpr (NB == 4 ? (METHOD == M_NEUMANN || (REFINE && METHOD != M_NEWTON_SCHULZ)) : (NB == 2 && METHOD == M_MIXED32 && OP == OP_F32 && REFINE)) {
        // the Neumann product wants every tile in both orientations, the refinement step most of them a second time (GlobalAnyA; the
        // same with the loads early or typed: C = 64, 32768 matrices, Neumann 460 against 505 us with fp32 operands, 117 against 126
        // with 16-bit ones and a 16-bit result; refinement after the blocked recursion 217 against 295 and 168 against 190, after the
        // direct leaves in fp32 207 against 279; b0 = 32 at C = 32 501 against 575.  Newton-Schulz reads A once, at C = 128 the
        // step is a kernel of its own, and at C = 32 the other methods hold all of A: 1.0 to 1.4 times as fast typed)
        invert_and_store<OP, NB, METHOD, GlobalAnyA<NB>, REFINE>(GlobalAnyA<NB>{static_cast<const char*>(A) + m * C * C * (in_dt == OP_F32 ? 4 : 2), in_dt, ln}, Tm, lds, ln, aux);
    } else if constexpr (REFINE || (METHOD == M_BLOCK_DIRECT && NB == 8)) {
        // tile by tile: the refinement step wants every tile once more, in both orientations; the direct leaves at C = 128 do
        // little enough before the merges to gain nothing from the early loads (84 us against 85, 4096 matrices)
        invert_and_store<OP, NB, METHOD, GlobalA<NB, IN>, REFINE>(GlobalA<NB, IN>{base, ln}, Tm, lds, ln, aux);
    } else {
        LoadedA<NB, METHOD> src;
        src.load(base, ln);
        invert_and_store<OP, NB, METHOD, LoadedA<NB, METHOD>, REFINE>(src, Tm, lds, ln, aux);
    }
}

// Workgroup -> matrix map of the fused kernels.  Workgroups are handed to the 8 XCDs round-robin
// (workgroup id mod 8); the H heads of one (batch, chunk) read the same beta / g cache lines, so
// they are given to one XCD, back to back, and share those lines in its L2.  Groups beyond the
// last multiple of 8 keep the identity map.
__device__ __forceinline__ int64_t head_group_swizzle(int64_t bid, int64_t n_group, int H)
{
    const int64_t full = (n_group / 8) * 8;
    if (bid >= full * H) return bid;
    const int64_t x = bid % 8, q = bid / 8;
    return ((q / H) * 8 + x) * H + (q % H);
}

// WPB wavefronts per workgroup, each with its own matrix.
// spread = 0 (many heads): wave w of workgroup u takes head unit * WPB + w of one (batch, chunk), so a workgroup reads
// WPB adjacent 256-byte key rows of every token (measured a few percent faster than one head per workgroup); falls back
// to the plain order when H is not a multiple of WPB.
// spread = S > 0 (few heads, H < 8: the layout a tensor-parallel shard sees): with the map above a workgroup's whole
// traffic would fall into one contiguous 64 KB stretch of K and one of T -- few memory channels at a time; measured 8-12 %
// slower, with 10 % higher read latency and 4.5x the DRAM credit stalls.  Instead a workgroup takes ONE head of WPB chunks
// S chunks apart (S = max(1, 4 / H), so its four key regions are at least 64 KB apart), and the S * H workgroups that share
// those 4 S chunks run back to back on one XCD.  Chunks beyond the last full group of 4 S keep the plain order.
// spread = ONE_WAVE_PER_GROUP (few matrices, see fused_grid): a workgroup has one matrix, in plain order.
// The waves never synchronise with each other.  Returns chunk id * H + head, or -1 for a wave without a matrix.
template <int WPB>
__device__ __forceinline__ int64_t fused_matrix_index(int64_t n_chunk, int H, int64_t n_mat, int spread)
{
    const int w = (WPB == 1) ? 0 : __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (WPB > 1 && spread > 0) {
        const int64_t per_group = (int64_t)spread * H;                 // workgroups per group of WPB * spread chunks
        const int64_t n_group = n_chunk / (WPB * spread);
        const int64_t full = n_group * per_group;
        const int64_t bid = blockIdx.x;
        if (bid < full) {
            const int64_t gh = head_group_swizzle(bid, n_group, (int)per_group);
            const int64_t grp = gh / per_group;
            const int r = (int)(gh - grp * per_group);                 // j * H + head, j = offset inside the stride
            const int64_t chunk = grp * (WPB * spread) + r / H + (int64_t)spread * w;
            return chunk * H + r % H;
        }
        const int64_t m = (full + (bid - full)) * WPB + w;             // the tail: WPB consecutive matrices per workgroup
        return m < n_mat ? m : -1;
    }
    if (H % WPB != 0 || (WPB > 1 && spread < 0)) {
        const int64_t m = WPB > 1 && spread < 0 ? (int64_t)blockIdx.x : (int64_t)blockIdx.x * WPB + w;
        return m < n_mat ? m : -1;
    }
    return head_group_swizzle(blockIdx.x, n_chunk, H / WPB) * WPB + w;
}

// The same for the fused kernels.  At C = 32 the Neumann product, and the direct leaves with fp32 operands, keep the patch that fits
// C = 128: it holds a compute unit to four workgroups, and the compiler then spends more registers on loads in flight.
// 32768 matrices of d_k = 128, bf16 keys, a patch of their own size / this: Neumann fp32 32.3 / 29.5 us, direct leaves 18.6 / 17.5;
// 131072, Neumann 16-bit 62 / 60, fp32 keys 138 / 126.  (Neumann, 16-bit operands, 64 fp32 channels: 0.92 times as fast with it.)
template <int KD, int OP, int NB, int METHOD, int DKS> constexpr int gdn_lds_floats()
{
    constexpr bool large = METHOD == M_NEUMANN ? !(OP != OP_F32 && KD == OP_F32 && DKS == 4) : METHOD == M_BLOCK_DIRECT && OP == OP_F32;
    return NB == 2 && large ? STORE_LDS_FLOATS : core_lds_floats<NB, METHOD>();
}

template <int KD, int OP, int NB, int METHOD, int DKS, bool REFINE = false, int WPB = 1>
__global__ __launch_bounds__(64 * WPB) __attribute__((amdgpu_waves_per_eu(min_waves_per_simd<OP, NB, METHOD, REFINE>()))) void k_gdn_tri_inv(const void* __restrict__ K, const float* __restrict__ beta,
                                                          const float* __restrict__ g, float* __restrict__ T,
                                                          uint32_t n_chunk, InvMapIf<gdn_lengths(16 * NB, KD, key_channels(KD, DKS), METHOD, REFINE)> map, int H, int d_k, uint8_t aux, uint8_t out_dt, int8_t spread)
{
    arguments_together(n_chunk, K, beta, g, T, map);
    constexpr int C = 16 * NB;
    constexpr int CORE = gdn_lds_floats<KD, OP, NB, METHOD, DKS>();
    constexpr int GATE = gate_lds_floats<NB>();
    constexpr int PER_WAVE = CORE > GATE ? CORE : GATE;
    __shared__ __attribute__((aligned(16))) float lds_all[WPB * PER_WAVE];
    float* lds = lds_all + ((WPB == 1) ? 0 : __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6))) * PER_WAVE;
    const int64_t m = fused_matrix_index<WPB>(n_chunk, H, n_chunk * H, spread);  // chunk id * H + h
    if (m < 0) return;
    const uint32_t bc = (uint32_t)m / (uint32_t)H;  // m < 2^31 (checked by the host)
    const int h = (int)((uint32_t)m - bc * (uint32_t)H);
    const ChunkPos pos = locate_chunk<C>(map, bc);
    const int64_t tok0 = pos.tok0;
    const Lane ln = lane_id();
    GramA<KD, NB, DKS> src;
    src.ln = ln;
    const int64_t esz = (KD == OP_F32) ? 4 : 2;
    src.issue_gate(beta + tok0 * H + h, g ? g + tok0 * H + h : nullptr, H, pos.valid);
    src.load_keys(static_cast<const char*>(K) + (tok0 * H + h) * (int64_t)d_k * esz, (int64_t)H * d_k, pos.valid);
    src.stage_gate(lds);
    invert_and_store<OP, NB, METHOD, GramA<KD, NB, DKS>, REFINE>(src, out_matrix(T, m, C, out_dt), lds, ln, aux);
}

// Fused kernel of the scalar / no-gate kinds for head dimensions without a specialised build.
// TEAM: the workgroup's wavefronts form a matrix together, its first one goes on alone (see Team; a kernel of its own: the other one lost 5 to
// 13 % of its speed with the choice at run time).
template <int KD, int OP, int NB, int METHOD, bool TEAM>
__global__ __launch_bounds__(TEAM ? 64 * TEAM_WAVES : 64) __attribute__((amdgpu_waves_per_eu(min_waves_per_simd<OP, NB, METHOD, false>()))) void k_gdn_any_dk_tri_inv(const void* __restrict__ K, const float* __restrict__ beta,
                                                           const float* __restrict__ g, float* __restrict__ T,
                                                           uint32_t n_chunk, InvMap map, int H, int d_k, uint8_t aux, uint8_t out_dt)
{
    arguments_together(n_chunk, K, beta, g, T, map);
    constexpr int C = 16 * NB;
    constexpr int CORE = core_lds_floats<NB, METHOD>();
    constexpr int GATE = gate_lds_floats<NB>();
    __shared__ __attribute__((aligned(16))) float lds[CORE > GATE ? CORE : GATE];
    __shared__ __attribute__((aligned(16))) char team_lds[TEAM ? team_lds_bytes<KD, NB, METHOD, false>() : 16];
    const int64_t m = head_group_swizzle(blockIdx.x, n_chunk, H);
    const uint32_t bc = (uint32_t)m / (uint32_t)H;
    const int h = (int)((uint32_t)m - bc * (uint32_t)H);
    const ChunkPos pos = locate_chunk<C>(map, bc);
    const int64_t tok0 = pos.tok0;
    const Lane ln = lane_id();
    const int64_t esz = (KD == OP_F32) ? 4 : 2;
    PreA<NB> src;
    if (!build_A_scalar_any_dk<KD, NB, METHOD, TEAM>(src, static_cast<const char*>(K) + (tok0 * H + h) * (int64_t)d_k * esz, (int64_t)H * d_k,
                                               beta + tok0 * H + h, g ? g + tok0 * H + h : nullptr, H, d_k, lds, ln, pos.valid,
                                               this_team(team_lds)))
        return;
    invert_and_store<OP, NB, METHOD, PreA<NB>, false>(src, out_matrix(T, m, C, out_dt), lds, ln, aux);
}

// Fused kernel for the per-channel gate: g is [B, Tlen, H, d_k]; the gated keys are rounded to OP.
// TEAM: WPB = 1, a workgroup of TEAM_WAVES wavefronts per matrix.
template <int OP, int NB, int METHOD, int WPB = 1, bool REFINE = false, bool TEAM = false>
__global__ __launch_bounds__(TEAM ? 64 * TEAM_WAVES : 64 * WPB) __attribute__((amdgpu_waves_per_eu(min_waves_per_simd<OP, NB, METHOD, REFINE, true>()))) void k_kda_tri_inv(const void* __restrict__ K, const float* __restrict__ beta,
                                                          const float* __restrict__ g, float* __restrict__ T,
                                                          uint32_t n_chunk, InvMapIf<kda_lengths(16 * NB, METHOD, REFINE)> map, int H, int d_k, uint8_t k_dt, uint8_t aux, uint8_t out_dt, int8_t spread)
{
    if constexpr (kda_lengths(16 * NB, METHOD, REFINE)) arguments_together(n_chunk, K, beta, g, T, map);
    constexpr int C = 16 * NB;
    constexpr int CORE = core_lds_floats<NB, METHOD>();
    constexpr int PER_WAVE = CORE > C ? CORE : C;
    __shared__ __attribute__((aligned(16))) float lds_all[WPB * PER_WAVE];
    float* lds = lds_all + ((WPB == 1) ? 0 : __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6))) * PER_WAVE;
    __shared__ __attribute__((aligned(16))) char team_lds[TEAM ? team_lds_bytes<OP, NB, REFINE ? METHOD + WITH_REFINE : METHOD, true>() : 16];
    const int64_t m = TEAM ? (int64_t)blockIdx.x : fused_matrix_index<WPB>(n_chunk, H, n_chunk * H, spread);
    if (m < 0) return;
    const uint32_t bc = (uint32_t)m / (uint32_t)H;
    const int h = (int)((uint32_t)m - bc * (uint32_t)H);
    const ChunkPos pos = locate_chunk<C>(map, bc);
    const int64_t tok0 = pos.tok0;
    const Lane ln = lane_id();
    const int64_t esz = (k_dt == OP_F32) ? 4 : 2;
    const int64_t e0 = (tok0 * H + h) * (int64_t)d_k;  // element offset of (token 0, head h, channel 0)
    PreA<NB> src;
    if (!build_A_per_channel<OP, NB, REFINE ? METHOD + WITH_REFINE : METHOD, TEAM>(src, static_cast<const char*>(K) + e0 * esz, k_dt, g + e0,
                                                                                   (int64_t)H * d_k, beta + tok0 * H + h, H, d_k, lds, ln, pos.valid,
                                                                                   n_chunk * H <= GATES_AHEAD_MATRICES, this_team(team_lds)))
        return;
    invert_and_store<OP, NB, METHOD, PreA<NB>, REFINE>(src, out_matrix(T, m, C, out_dt), lds, ln, aux);
}

// ---------------------------------------------------------------------------------------------
// C = 128 on one workgroup of four wavefronts per matrix (Neumann product, Newton-Schulz, refinement pass):
// wave w owns tile rows w and 7 - w of every matrix involved.  The refinement pass keeps its Y in LDS as 36 fp32
// tiles (16 x 20 floats each), readable in either orientation.
// ---------------------------------------------------------------------------------------------
constexpr int N128_NB = 8;
constexpr int N128_NT = 36;
constexpr int N128_LDS_FLOATS = N128_NT * XPOSE_FLOATS;   // 46 080 bytes

__device__ __forceinline__ v4f lds_tile_read_n(const float* t, Lane ln)
{
    v4f v;
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = t[(4 * ln.q + r) * XPOSE_LD + ln.n];
    return v;
}
// slot s of wave W: tile (i, j) with i = W for s <= W, else i = 7 - W
template <int W> __host__ __device__ constexpr int n128_row(int s) { return s <= W ? W : 7 - W; }
template <int W> __host__ __device__ constexpr int n128_col(int s) { return s <= W ? s : s - (W + 1); }

template <int W, bool IS_T = true>
__device__ __forceinline__ void n128_store(Out Tm, const v4f (&Xt)[9], float* patch, Lane ln)
{
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        const int i = half == 0 ? W : 7 - W, s0 = half == 0 ? 0 : W + 1;
        v4f row[N128_NB];
#pragma unroll
        for (int j = 0; j < N128_NB; ++j)
            if (j <= i) row[j] = Xt[s0 + j];
        store_strip<N128_NB>(Tm, i, row, [](int) { return IS_T; }, patch, ln);
    }
}

#define TRIINV_PER_WAVE(w, CALL) \
    switch (w) {                 \
    case 0: { constexpr int W = 0; CALL; } break; \
    case 1: { constexpr int W = 1; CALL; } break; \
    case 2: { constexpr int W = 2; CALL; } break; \
    default: { constexpr int W = 3; CALL; } break; \
    }

// Eight wavefronts: two to a pair of tile rows, one for the even tile columns and one for the odd (Newton-Schulz, few matrices).  The two that share a
// SIMD, w and w + 4, have 29 to 31 of a product's 120 tile products between them, the longest 21 (of four wavefronts 25 to 37).
#define TRIINV_PER_HALF_WAVE(w, CALL) \
    switch (w) {                      \
    case 0: { constexpr int W = 0, PART = 0; CALL; } break; \
    case 1: { constexpr int W = 0, PART = 1; CALL; } break; \
    case 2: { constexpr int W = 1, PART = 0; CALL; } break; \
    case 3: { constexpr int W = 1, PART = 1; CALL; } break; \
    case 4: { constexpr int W = 3, PART = 1; CALL; } break; \
    case 5: { constexpr int W = 3, PART = 0; CALL; } break; \
    case 6: { constexpr int W = 2, PART = 1; CALL; } break; \
    default: { constexpr int W = 2, PART = 0; CALL; } break; \
    }
// Its W.
__device__ __forceinline__ int n128_pair(int w) { return w < 4 ? w >> 1 : 5 - (w >> 1); }

// ---------------------------------------------------------------------------------------------
// Newton-Schulz at C = 128 (paper Alg. 3, Eq. 8, for I + A): the same four-wavefront workgroup (few matrices: eight, see TRIINV_PER_HALF_WAVE).
//   X <- I / C;  n_iter times:  Y <- X + A X;  X <- 2 X - X Y.
// Wave w owns tile rows w and 7 - w: it keeps its rows of A (T orientation, packed operands) and of X (N
// orientation, fp32) in registers and reads the right factor of every product (a tile of X, then of Y, in N
// orientation) from LDS, and X's left form, turned, from its own tiles there (TurnTiles).  The rounding to the
// operand type happens once, at the writer.  X and Y take 2 x 36 tiles, 36 KB, with 16-bit operands; fp32 ones, split in three, take turns on 54 KB.
// ---------------------------------------------------------------------------------------------
// The tiles of the Neumann product below.  A right factor in N orientation is exactly the register image its producer holds,
// so a tile crosses between waves as a mailbox: 64 consecutive slots of one packed operand each, lane l of the
// reader taking what lane l of the writer left.  No transposition, no bank conflicts.
template <int OP> struct MailTiles {
    static constexpr int TILE_BYTES = 64 * (int)sizeof(Opnd<OP>);
    static constexpr int BYTES = N128_NT * TILE_BYTES;
    static __device__ __forceinline__ void put(char* base, int tile, Opnd<OP> v, Lane ln)
    {
        *reinterpret_cast<Opnd<OP>*>(base + tile * TILE_BYTES + (16 * ln.q + ln.n) * (int)sizeof(Opnd<OP>)) = v;
    }
    static __device__ __forceinline__ Opnd<OP> get(const char* base, int tile, Lane ln)
    {
        return *reinterpret_cast<const Opnd<OP>*>(base + tile * TILE_BYTES + (16 * ln.q + ln.n) * (int)sizeof(Opnd<OP>));
    }
};

// Two sets of tiles, later the four store patches.
template <int OP> constexpr int mail128_lds_bytes()
{
    return 2 * MailTiles<OP>::BYTES > 4 * STORE_LDS_FLOATS * 4 ? 2 * MailTiles<OP>::BYTES : 4 * STORE_LDS_FLOATS * 4;
}

// The tiles of Newton-Schulz: each part of a tile (fp32 operands: the three of Split3) in the order of Turn16, so that it is read as it was
// written, by any wave, or transposed.
template <int OP> struct TurnTiles {
    static constexpr int PARTS = OP == OP_F32 ? 3 : 1;
    static constexpr int BYTES = N128_NT * PARTS * TURN16_BYTES;
    Turn16 at;
    __device__ __forceinline__ TurnTiles(char* base, Lane ln) : at(reinterpret_cast<float*>(base), ln) {}
    __device__ __forceinline__ void put(int tile, int part, v2u u) const { at.put(tile * PARTS + part, u); }
    template <bool TR> __device__ __forceinline__ v2u get(int tile, int part) const
    {
        return TR ? at.get(tile * PARTS + part) : *reinterpret_cast<const v2u*>(at.put_at + (tile * PARTS + part) * TURN16_BYTES);
    }
};
// X and Y: 16-bit operands a set each, fp32 ones a set for both in turns (a second one of 54 KB would leave a compute unit one workgroup).
// Later the store patches; eight wavefronts: all eight strips of the result.
constexpr int NS128_STRIP_LD = 128 + 4;
template <int OP, int WAVES = 4> constexpr int ns128_lds_bytes()
{
    constexpr int tiles = (OP == OP_F32 ? 1 : 2) * TurnTiles<OP>::BYTES, store = WAVES == 8 ? 128 * NS128_STRIP_LD * 4 : 4 * STORE_LDS_FLOATS * 4;
    return tiles > store ? tiles : store;
}

template <int W> __host__ __device__ constexpr int n128_slot(int i, int k) { return i == W ? k : (W + 1) + k; }

// The wave's two tile rows as left operands, and one tile column as right operand.  16-bit operands: pairs of tiles for the
// 32-deep instructions; fp32: tile by tile, each split into three bf16 parts (see Split3).
template <int OP> struct Ns128Operands {
    static constexpr float SCALE = 1.f;  // of X and Y
    typedef PairOp<OP> Row[4];
    static __device__ __forceinline__ void put(Row& row, int k, Opnd<OP> x) { row[k / 2].set(k & 1, x); }
    template <bool TR> static __device__ __forceinline__ void get(Row& row, int k, const TurnTiles<OP>& tiles, int tile)
    {
        Opnd<OP> o;
        o.x = __builtin_bit_cast(decltype(o.x), tiles.template get<TR>(tile, 0));
        put(row, k, o);
    }
    static __device__ __forceinline__ void publish(const TurnTiles<OP>& tiles, int tile, v4f x)
    {
        tiles.put(tile, 0, __builtin_bit_cast(v2u, pack<OP>(x).x));
    }
    // acc[h] += sum over k of l[h](k) times tile (k, j) of the tiles, for the rows i = W and 7 - W that have a column j
    template <int W> static __device__ __forceinline__ void products(const Row (&l)[2], const TurnTiles<OP>& tiles, int j, v4f (&acc)[2])
    {
        Row r;
#pragma unroll
        for (int k = 0; k < N128_NB; ++k)
            if (k >= j && k <= 7 - W) get<false>(r, k, tiles, tix(k, j));
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int i = h == 0 ? W : 7 - W;
            if (j > i) continue;
            v4f odd;
#pragma unroll
            for (int p = 0; p < 4; ++p) pair_term<OP>(p, i, j, l[h][p], r[p], acc[h], odd);
            if (mixed_terms(i, j)) acc[h] += odd;
        }
    }
};
template <> struct Ns128Operands<OP_F32> {
    // Halved: the leading part of a split tile is up to 2^-8 larger than the tile and infinite from 3.396e38 on, where the iterate is finite.
    static constexpr float SCALE = 0.5f;
    typedef Split3 Row[8];
    static __device__ __forceinline__ void put(Row& row, int k, Opnd<OP_F32> x) { row[k] = split3_any(x.x); }
    template <bool TR> static __device__ __forceinline__ void get(Row& row, int k, const TurnTiles<OP_F32>& tiles, int tile)
    {
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            const v2u u = tiles.get<TR>(tile, p);
            row[k].u[2 * p] = u[0];
            row[k].u[2 * p + 1] = u[1];
        }
    }
    static __device__ __forceinline__ void publish(const TurnTiles<OP_F32>& tiles, int tile, v4f x)
    {
        const Split3 s = split3(x);
#pragma unroll
        for (int p = 0; p < 3; ++p) tiles.put(tile, p, v2u{s.u[2 * p], s.u[2 * p + 1]});
    }
    template <int W> static __device__ __forceinline__ void products(const Row (&l)[2], const TurnTiles<OP_F32>& tiles, int j, v4f (&acc)[2])
    {
        v4f cross[2] = {zero4(), zero4()};
#pragma unroll
        for (int k = 0; k < N128_NB; ++k) {
            if (k < j || k > 7 - W) continue;
            Row r;
            get<false>(r, k, tiles, tix(k, j));
#pragma unroll
            for (int part = 0; part < 3; ++part)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    if (k > (h == 0 ? W : 7 - W)) continue;
                    if (part < 2)
                        cross[h] = tn_split(part, l[h][k], r[k], cross[h]);
                    else
                        acc[h] = tn_split(part, l[h][k], r[k], acc[h]);
                }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
            if (j <= (h == 0 ? W : 7 - W)) acc[h] += cross[h];
    }
};

// The transpose of a tile, exact (see Split3; for values beyond the largest bf16 too): by products with the identity.
template <int OP> __device__ __forceinline__ v4f turned(Opnd<OP> x, Opnd<OP_BF16> id_bf16, Opnd<OP> id)
{
    if constexpr (OP == OP_F32) {
        const Split3 s = split3_any(x.x);
        return tn<OP_BF16>(s.h(), id_bf16, tn<OP_BF16>(s.m(), id_bf16, tn<OP_BF16>(s.l(), id_bf16, zero4())));
    } else {
        return tn<OP>(x, id, zero4());
    }
}

// At: this wave's nine tiles of A in T orientation (slot order of n128_row / n128_col).  lds: ns128_lds_bytes<OP>() bytes
// that no wave uses for anything else any more.
// X is kept in N orientation only; its left form is read back from the wave's own tiles in LDS by transposing reads; a tile column of the
// right factor is read from LDS once for both of the wave's rows; 16-bit operands contract two tiles per instruction, fp32 ones are split
// into three bf16 parts; the first iteration from I / C is a scaling.
// Bound by latency: LDS reads a column at a time and two (fp32: four) barriers an iteration.  1024 fused matrices with fp32 operands, by fp32
// instructions / split 245.1 / 182.3 us, standalone 239.4 / 179.1, 16 of them 73 / 71 (by eight wavefronts 50; a fiftieth of each for the halving), error
// against 64 bits at most that of fp32 instructions for every gate, head dimension and key type: 1.33e-7 / 1.31e-7 (standalone 8.6e-8 / 5.8e-8, correlated
// keys 3.75e-7 / 3.70e-7, per-channel gate 2.34e-7 / 2.33e-7).  Iterates below 2^-109 lose low bits that fp32 instructions keep.
// X turned by products with the identity / by LDS reads: 4096 bf16 188 / 173, 2048 standalone 96 / 86.
// PART: 0, 1: of eight wavefronts, this one's columns are the even / odd ones (TRIINV_PER_HALF_WAVE); -1: all.
template <int OP, int W, int PART = -1>
__device__ __forceinline__ void ns128_run(const Opnd<OP> (&At)[9], Out Tm, char* lds, Lane ln, int n_iter, int w)
{
    typedef Ns128Operands<OP> Ops;
    constexpr bool ONE_SET = OP == OP_F32;
    constexpr int ROW[2] = {W, 7 - W};
    constexpr float X0 = 1.f / 128.f;
    constexpr auto mine = [](int j) { return PART < 0 || (j & 1) == PART; };
    const TurnTiles<OP> X(lds, ln), Y(lds + (ONE_SET ? 0 : TurnTiles<OP>::BYTES), ln);
    const v4f unit = identity_tile(ln);
    typename Ops::Row Al[2];
    v4f Xn[9];
    {
        const Opnd<OP> id = pack<OP>(unit);
        const Opnd<OP_BF16> id_bf16 = pack<OP_BF16>(unit);
#pragma unroll
        for (int s = 0; s < 9; ++s) {
            const int i = n128_row<W>(s), j = n128_col<W>(s);
            Ops::put(Al[s <= W ? 0 : 1], j, At[s]);
            if (!mine(j)) continue;
            v4f a = turned<OP>(At[s], id_bf16, id);
            if (i == j) a += unit;
            Xn[s] = Ops::SCALE * ((i == j ? 2.f * X0 : 0.f) * unit - X0 * X0 * a);
            Ops::publish(X, tix(i, j), Xn[s]);
        }
    }
    __syncthreads();
#pragma unroll 1
    for (int it = 1; it < n_iter; ++it) {
        // Y(i,j) = X(i,j) + sum_k A(i,k) X(k,j) on this wave's rows
        v4f Yn[9];
#pragma unroll
        for (int j = 0; j <= 7 - W; ++j) {
            if (!mine(j)) continue;
            v4f y[2];
#pragma unroll
            for (int h = 0; h < 2; ++h)
                if (j <= ROW[h]) y[h] = Xn[n128_slot<W>(ROW[h], j)];
            Ops::template products<W>(Al, X, j, y);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (j > ROW[h]) continue;
                if (ONE_SET)
                    Yn[n128_slot<W>(ROW[h], j)] = y[h];
                else
                    Ops::publish(Y, tix(ROW[h], j), y[h]);
            }
            __builtin_amdgcn_sched_barrier(0);  // (the next column's tiles and X's left form would not fit beside this one's)
        }
        typename Ops::Row Xl[2];
#pragma unroll
        for (int s = 0; s < 9; ++s) Ops::template get<true>(Xl[s <= W ? 0 : 1], n128_col<W>(s), X, tix(n128_row<W>(s), n128_col<W>(s)));
        __syncthreads();  // nobody reads X from LDS any more in this iteration; two sets: Y complete
        if (ONE_SET) {
#pragma unroll
            for (int s = 0; s < 9; ++s)
                if (mine(n128_col<W>(s))) Ops::publish(Y, tix(n128_row<W>(s), n128_col<W>(s)), Yn[s]);
            __syncthreads();  // Y complete
        }
        // X(i,j) <- 2 X(i,j) - sum_k X(i,k) Y(k,j)
#pragma unroll
        for (int j = 0; j <= 7 - W; ++j) {
            if (!mine(j)) continue;
            v4f xy[2] = {zero4(), zero4()};
            Ops::template products<W>(Xl, Y, j, xy);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (j > ROW[h]) continue;
                const int s = n128_slot<W>(ROW[h], j);
                if constexpr (Ops::SCALE == 1.f) {
                    Xn[s] = 2.f * Xn[s] - xy[h];
                } else {  // 2 X and X Y may overflow where their difference does not; the same rounding
                    static_assert(Ops::SCALE == 0.5f, "X and Y in halves");
                    const v4f d = Xn[s] - xy[h];
                    Xn[s] = d + d;
                }
                if (!ONE_SET) Ops::publish(X, tix(ROW[h], j), Xn[s]);
            }
            if (ONE_SET) __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();  // nobody reads Y any more; two sets: X complete
        if (ONE_SET && it + 1 < n_iter) {
#pragma unroll
            for (int s = 0; s < 9; ++s)
                if (mine(n128_col<W>(s))) Ops::publish(X, tix(n128_row<W>(s), n128_col<W>(s)), Xn[s]);
            __syncthreads();  // X complete
        }
    }
#pragma unroll
    for (int s = 0; s < 9; ++s)
        if (mine(n128_col<W>(s))) Xn[s] *= 1.f / Ops::SCALE;
    // X and Y in LDS are dead: their memory becomes the four store patches, or the strips of the whole result
    if constexpr (PART < 0) {
        n128_store<W, false>(Tm, Xn, reinterpret_cast<float*>(lds) + w * STORE_LDS_FLOATS, ln);
    } else {
        float* const strips = reinterpret_cast<float*>(lds);
#pragma unroll
        for (int s = 0; s < 9; ++s) {
            const int i = n128_row<W>(s), j = n128_col<W>(s);
            if (mine(j)) strip_tile<NS128_STRIP_LD>(strips + i * 16 * NS128_STRIP_LD, i, j, Xn[s], false, ln);
        }
        __syncthreads();
        flush_strip<N128_NB, false, NS128_STRIP_LD>(Tm, w, strips + w * 16 * NS128_STRIP_LD, ln);
    }
}

// The fused kernel's tiles of A: the four waves load the chunk's keys once between them (wave w its tile rows w and
// 7 - w), pass them through LDS in mailbox form (slot [tile row][k-step][lane], one 16-byte
// key vector each) and every wave forms only its own nine tiles.
template <int KD, int DKS, int ROWS = 2> struct SharedKeys128 {
    typedef typename KeyVec<KD>::type kvec;
    static constexpr int KSTEP = (KD == OP_F32) ? 16 : 32;
    static constexpr int BYTES = 8 * DKS * 64 * 16;
    kvec own[ROWS][DKS];  // ROWS = 2: tile rows w and 7 - w, 1: w

    // Kc: first key element of (chunk row 0, this head); row_stride in elements; rows beyond valid read the last real token and become zero.
    __device__ __forceinline__ void load(const void* Kc, int64_t row_stride, int valid, int w, Lane ln)
    {
        constexpr int per_lane = (KD == OP_F32) ? 4 : 8;
        const kvec zero = __builtin_bit_cast(kvec, v4u{0u, 0u, 0u, 0u});
#pragma unroll
        for (int h = 0; h < ROWS; ++h)
#pragma unroll
            for (int s = 0; s < DKS; ++s) {
                const int row = 16 * (h == 0 ? w : 7 - w) + ln.n;
                const int64_t off = (int64_t)(row < valid ? row : valid - 1) * row_stride + KSTEP * s + per_lane * ln.q;
                kvec v;
                if (KD == OP_F32)
                    v = *reinterpret_cast<const kvec*>(static_cast<const float*>(Kc) + off);
                else
                    v = *reinterpret_cast<const kvec*>(static_cast<const uint16_t*>(Kc) + off);
                own[h][s] = row < valid ? v : zero;
            }
    }
    __device__ __forceinline__ void publish(char* lds, int w, Lane ln) const
    {
#pragma unroll
        for (int h = 0; h < ROWS; ++h)
#pragma unroll
            for (int s = 0; s < DKS; ++s)
                *reinterpret_cast<kvec*>(lds + (((h == 0 ? w : 7 - w) * DKS + s) * 64 + 16 * ln.q + ln.n) * 16) = own[h][s];
    }
    // Tile s of wave W (slot order of n128_row / n128_col) in N (TR = false) or T orientation; after a barrier that
    // follows every wave's publish().
    template <int W, bool TR>
    __device__ __forceinline__ v4f tile(const char* lds, const GateVec<N128_NB>& gate, int s, Lane ln) const
    {
        const int i = n128_row<W>(s), j = n128_col<W>(s);
        v4f acc = zero4();
#pragma unroll
        for (int t = 0; t < DKS; ++t) {
            // both from LDS: the loaded keys' registers are free again once they are published
            const kvec kj = *reinterpret_cast<const kvec*>(lds + ((j * DKS + t) * 64 + 16 * ln.q + ln.n) * 16);
            const kvec ki = *reinterpret_cast<const kvec*>(lds + ((i * DKS + t) * 64 + 16 * ln.q + ln.n) * 16);
            acc = TR ? gram_step<KD>(kj, ki, acc) : gram_step<KD>(ki, kj, acc);
        }
        return gate.template apply<TR>(i, j, acc, ln);
    }
};

// SharedKeys128 behind the tile-source interface, for the tiles of wave W only.
template <int KD, int DKS, int W, int ROWS = 2> struct SharedA128 {
    const SharedKeys128<KD, DKS, ROWS>& keys;
    const GateVec<N128_NB>& gate;
    const char* lds;
    Lane ln;
    template <bool TR> __device__ __forceinline__ v4f get(int i, int j) const
    {
        return keys.template tile<W, TR>(lds, gate, i == W ? j : (W + 1) + j, ln);
    }
};

template <int OP, int W, class ASrc> __device__ __forceinline__ void ns128_tiles_of(const ASrc& A, Opnd<OP> (&At)[9])
{
#pragma unroll
    for (int s = 0; s < 9; ++s) At[s] = pack<OP>(A.template get<true>(n128_row<W>(s), n128_col<W>(s)));
}

// ---------------------------------------------------------------------------------------------
// Neumann product at C = 128, (I + A)^-1 = (I - A) (I + A^2) (I + A^4) ... (I + A^64): the four-wavefront workgroup
// and mailbox tiles (MailTiles).  Wave w owns tile rows w and 7 - w.  It keeps X^T (fp32)
// and its rows of the running power Y = A^(2^k) in T orientation (packed) in registers; every product takes its
// other factor, a tile of Y in N orientation, from the mailbox.  Squaring forms both orientations of the new tile
// (two matrix-core instructions per product instead of one transposing read through LDS); the N image goes to the
// other of two mailbox buffers, which leaves one barrier per iteration:
//   Y' <- Y Y (cur -> nxt);  barrier;  X^T += Y'^T X^T (reads nxt);  swap.
// ---------------------------------------------------------------------------------------------
// Wave W's share of the start: X^T = I - A^T and Y = A in T orientation into registers, Y in N orientation into the mailbox.
template <int OP, int W, class ASrc>
__device__ __forceinline__ void neumann128_prepare(const ASrc& A, v4f (&Xt)[9], Opnd<OP> (&yt)[9], char* cur, Lane ln)
{
#pragma unroll
    for (int s = 0; s < 9; ++s) {
        const int i = n128_row<W>(s), j = n128_col<W>(s);
        MailTiles<OP>::put(cur, tix(i, j), pack<OP>(A.template get<false>(i, j)), ln);
        const v4f at = A.template get<true>(i, j);
#pragma unroll
        for (int r = 0; r < 4; ++r) Xt[s][r] = ((i == j && 4 * ln.q + r == ln.n) ? 1.f : 0.f) - at[r];
        yt[s] = pack<OP>(at);
    }
}

// cur, nxt: the two mailbox buffers (MailTiles<OP>::BYTES each), cur filled by neumann128_prepare; patch: this wave's
// store patch, anywhere in LDS that no wave uses for anything but the two buffers.
template <int OP, int W>
__device__ __forceinline__ void neumann128_run(v4f (&Xt)[9], Opnd<OP> (&yt)[9], Out Tm, char* cur, char* nxt, float* patch, Lane ln)
{
    typedef MailTiles<OP> Mail;
    __syncthreads();
#pragma unroll 1
    for (int it = 0; it < 6; ++it) {  // log2(128 / 2)
        const int p = 1 << it, pn = 2 << it;
        Opnd<OP> ytn[9];
#pragma unroll
        for (int s = 0; s < 9; ++s) {
            const int i = n128_row<W>(s), j = n128_col<W>(s);
            // structural zeros of A^p (tile (a, b) vanishes when 16 (a - b) + 15 < p); p is uniform
            const auto live = [&](int k) { return 16 * (i - k) + 15 >= p && 16 * (k - j) + 15 >= p; };
            const auto mine = [&](int k) { return yt[n128_slot<W>(i, k)]; };
            Opnd<OP> y[N128_NB];
#pragma unroll
            for (int k = 0; k < N128_NB; ++k)
                if (k >= j && k <= i) y[k] = Mail::get(cur, tix(k, j), ln);
            const auto theirs = [&](int k) { return y[k]; };
            const v4f an = tn_sum_if<OP>(j, i, mine, theirs, live, zero4());
            const v4f at = tn_sum_if<OP>(j, i, theirs, mine, live, zero4());
            ytn[s] = pack<OP>(at);
            Mail::put(nxt, tix(i, j), pack<OP>(an), ln);
        }
#pragma unroll
        for (int s = 0; s < 9; ++s) yt[s] = ytn[s];
        __syncthreads();  // the new power is complete; nobody reads the old one any more
        // X^T(i,j) += sum_k Y(k,j)^T X(i,k)^T over this wave's two tile rows; the packed old row first
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int i = half == 0 ? W : 7 - W, s0 = half == 0 ? 0 : W + 1;
            Opnd<OP> xo[N128_NB];
#pragma unroll
            for (int k = 0; k < N128_NB; ++k)
                if (k <= i) xo[k] = pack<OP>(Xt[s0 + k]);
#pragma unroll
            for (int j = 0; j < N128_NB; ++j) {
                if (j > i) continue;
                Xt[s0 + j] = tn_sum_if<OP>(
                    j, i, [&](int k) { return Mail::get(nxt, tix(k, j), ln); }, [&](int k) { return xo[k]; },
                    [&](int k) { return 16 * (k - j) + 15 >= pn; }, Xt[s0 + j]);
            }
        }
        char* const t = cur;
        cur = nxt;
        nxt = t;
    }
    __syncthreads();  // both mailbox buffers are dead: their memory becomes the four store patches
    n128_store<W>(Tm, Xt, patch, ln);
}

// ---------------------------------------------------------------------------------------------
// One step of iterative refinement at C = 128 (paper Alg. 6, Eq. 9, for I + A), as a second pass over
// a result Y that an earlier kernel left in T (fp32), in place:
//   R <- I - Y (I + A);   X <- Y + R Y.
// The same four-wavefront workgroup: Y goes to LDS (36 fp32 tiles, N layout); wave w keeps its tile
// rows w and 7 - w of Y^T and R^T in registers and forms
//   R^T(i,j) = [i==j] I - Y^T(i,j) - sum_k A(k,j)^T Y(i,k)^T,     X^T(i,j) = Y^T(i,j) + sum_k Y(k,j)^T R(i,k)^T.
// A wave reads and writes only its own rows of T in global memory, so the pass is safe in place.
// ---------------------------------------------------------------------------------------------
// Tile (k, j) of A as a left factor (N orientation, packed): formed on the spot by the sources that hold keys or read memory.
template <int OP, class ASrc> __device__ __forceinline__ Opnd<OP> left_operand(const ASrc& A, int k, int j)
{
    return pack<OP>(A.template get<false>(k, j));
}

template <int OP, int W, class ASrc>
__device__ __forceinline__ void refine128_run(const ASrc& A, float* Tm, float* Y, Lane ln, int w)
{
    v4f Yt[9];
#pragma unroll
    for (int s = 0; s < 9; ++s) {
        const int i = n128_row<W>(s), j = n128_col<W>(s);
        // row-major 16-byte pieces = the tile in T orientation: v[r] = Y[16i + n][16j + 4q + r]
        Yt[s] = *reinterpret_cast<const v4f*>(Tm + (16 * i + ln.n) * 128 + 16 * j + 4 * ln.q);
        *reinterpret_cast<v4f*>(&Y[tix(i, j) * XPOSE_FLOATS + ln.n * XPOSE_LD + 4 * ln.q]) = Yt[s];
    }
    __syncthreads();
    Opnd<OP> Rt[9];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        const int i = half == 0 ? W : 7 - W, s0 = half == 0 ? 0 : W + 1;
        Opnd<OP> yo[N128_NB];
#pragma unroll
        for (int k = 0; k < N128_NB; ++k)
            if (k <= i) yo[k] = pack<OP>(Yt[s0 + k]);
#pragma unroll
        for (int j = 0; j < N128_NB; ++j) {
            if (j > i) continue;
            v4f acc = zero4();
#pragma unroll
            for (int k = 0; k < N128_NB; ++k) {
                if (k < j || k > i) continue;
                acc = tn<OP>(left_operand<OP>(A, k, j), yo[k], acc);
            }
            v4f r;
#pragma unroll
            for (int e = 0; e < 4; ++e) r[e] = ((i == j && 4 * ln.q + e == ln.n) ? 1.f : 0.f) - Yt[s0 + j][e] - acc[e];
            Rt[s0 + j] = pack<OP>(r);
        }
    }
    v4f Xt[9];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        const int i = half == 0 ? W : 7 - W, s0 = half == 0 ? 0 : W + 1;
#pragma unroll
        for (int j = 0; j < N128_NB; ++j) {
            if (j > i) continue;
            v4f acc = Yt[s0 + j];
#pragma unroll
            for (int k = 0; k < N128_NB; ++k) {
                if (k < j || k > i) continue;
                acc = tn<OP>(pack<OP>(lds_tile_read_n(Y + tix(k, j) * XPOSE_FLOATS, ln)), Rt[s0 + k], acc);
            }
            Xt[s0 + j] = acc;
        }
    }
    __syncthreads();  // Y is dead: its memory becomes the four store patches
    n128_store<W>(Out{Tm, OP_F32}, Xt, Y + w * STORE_LDS_FLOATS, ln);
}

template <int IN, int OP>
__global__ __launch_bounds__(256) void k_tri_inv_refine128(const void* __restrict__ A, float* T, int64_t n_mat)
{
    __shared__ __attribute__((aligned(16))) float Y[N128_LDS_FLOATS];
    const int64_t m = blockIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const Lane ln = lane_id();
    const GlobalA<N128_NB, IN> src{static_cast<const char*>(A) + m * 128 * 128 * (IN == OP_F32 ? 4 : 2), ln};
    (void)n_mat;
    TRIINV_PER_WAVE(w, (refine128_run<OP, W>(src, T + m * 128 * 128, Y, ln, w)))
}

template <int KD, int OP, int DKS>
__global__ __launch_bounds__(256) void k_gdn_tri_inv_refine128(const void* __restrict__ K, const float* __restrict__ beta,
                                                               const float* __restrict__ g, float* T, uint32_t n_chunk,
                                                               InvMap map, int H, int d_k)
{
    arguments_together(n_chunk, K, beta, g, T, map);
    constexpr int C = 128;
    __shared__ __attribute__((aligned(16))) float Y[N128_LDS_FLOATS];
    const int64_t m = head_group_swizzle(blockIdx.x, n_chunk, H);
    const uint32_t bc = (uint32_t)m / (uint32_t)H;
    const int h = (int)((uint32_t)m - bc * (uint32_t)H);
    const ChunkPos pos = locate_chunk<C>(map, bc);
    const int64_t tok0 = pos.tok0;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const Lane ln = lane_id();
    GramA<KD, N128_NB, DKS> src;
    src.ln = ln;
    const int64_t esz = (KD == OP_F32) ? 4 : 2;
    src.issue_gate(beta + tok0 * H + h, g ? g + tok0 * H + h : nullptr, H, pos.valid);
    src.load_keys(static_cast<const char*>(K) + (tok0 * H + h) * (int64_t)d_k * esz, (int64_t)H * d_k, pos.valid);
    src.stage_gate(Y + w * 2 * C);  // a private 2 * C floats inside the (not yet used) Y buffer
    __syncthreads();
    TRIINV_PER_WAVE(w, (refine128_run<OP, W>(src, T + m * C * C, Y, ln, w)))
}

// WAVES: 4 or 8.
template <int IN, int OP, int WAVES = 4>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(WAVES == 8 || OP == OP_F32 ? 2 : 3))) void k_tri_inv_ns128(const void* A, float* T, int64_t n_mat, int n_iter, int out_dt)  // may run in place
{
    __shared__ __attribute__((aligned(16))) char lds[ns128_lds_bytes<OP, WAVES>()];
    const int64_t m = blockIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const Lane ln = lane_id();
    const GlobalA<N128_NB, IN> src{static_cast<const char*>(A) + m * 128 * 128 * (IN == OP_F32 ? 4 : 2), ln};
    (void)n_mat;
    Opnd<OP> At[9];
    // in place: every wave has read its tiles of A before any wave stores (a barrier lies between)
    if constexpr (WAVES == 8) {
        TRIINV_PER_HALF_WAVE(w, (ns128_tiles_of<OP, W>(src, At), ns128_run<OP, W, PART>(At, out_matrix(T, m, 128, out_dt), lds, ln, n_iter, w)))
    } else {
        TRIINV_PER_WAVE(w, (ns128_tiles_of<OP, W>(src, At)))
        TRIINV_PER_WAVE(w, (ns128_run<OP, W>(At, out_matrix(T, m, 128, out_dt), lds, ln, n_iter, w)))
    }
}

template <int KD, int OP, int DKS, int WAVES = 4>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(WAVES == 8 || OP == OP_F32 ? 2 : 3))) void k_gdn_tri_inv_ns128(const void* __restrict__ K, const float* __restrict__ beta,
                                                           const float* __restrict__ g, float* __restrict__ T,
                                                           uint32_t n_chunk, InvMap map, int H, int d_k, uint8_t n_iter, uint8_t out_dt)
{
    arguments_together(n_chunk, K, beta, g, T, map);
    constexpr int C = 128;
    typedef SharedKeys128<KD, DKS, 8 / WAVES> Keys;
    constexpr int GATE_BYTES = WAVES * 2 * C * 4;  // beta and g of the chunk, staged by every wave for itself
    constexpr int LDS_BYTES = ns128_lds_bytes<OP, WAVES>() > Keys::BYTES + GATE_BYTES ? ns128_lds_bytes<OP, WAVES>() : Keys::BYTES + GATE_BYTES;
    __shared__ __attribute__((aligned(16))) char lds[LDS_BYTES];
    const int64_t m = head_group_swizzle(blockIdx.x, n_chunk, H);
    const uint32_t bc = (uint32_t)m / (uint32_t)H;
    const int h = (int)((uint32_t)m - bc * (uint32_t)H);
    const ChunkPos pos = locate_chunk<C>(map, bc);
    const int64_t tok0 = pos.tok0;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const Lane ln = lane_id();
    const int64_t esz = (KD == OP_F32) ? 4 : 2;
    GateVec<N128_NB> gate;
    Keys keys;
    gate.issue(beta + tok0 * H + h, g ? g + tok0 * H + h : nullptr, H, ln, pos.valid);
    keys.load(static_cast<const char*>(K) + (tok0 * H + h) * (int64_t)d_k * esz, (int64_t)H * d_k, pos.valid, w, ln);
    gate.stage(reinterpret_cast<float*>(lds + Keys::BYTES) + w * 2 * C, ln);
    keys.publish(lds, w, ln);
    __syncthreads();
    Opnd<OP> At[9];
    if constexpr (WAVES == 8) {
        TRIINV_PER_HALF_WAVE(w, (ns128_tiles_of<OP, W>(SharedA128<KD, DKS, W, 1>{keys, gate, lds, ln}, At), __syncthreads(),
                                 ns128_run<OP, W, PART>(At, out_matrix(T, m, C, out_dt), lds, ln, n_iter, w)))
    } else {
        TRIINV_PER_WAVE(w, (ns128_tiles_of<OP, W>(SharedA128<KD, DKS, W>{keys, gate, lds, ln}, At)))
        __syncthreads();  // the keys in LDS are dead: X and Y take their place
        TRIINV_PER_WAVE(w, (ns128_run<OP, W>(At, out_matrix(T, m, C, out_dt), lds, ln, n_iter, w)))
    }
}

template <int IN, int OP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(OP == OP_F32 ? 2 : 3))) void k_tri_inv_neumann128(const void* A, float* T, int64_t n_mat, int out_dt)  // may run in place
{
    __shared__ __attribute__((aligned(16))) char lds[mail128_lds_bytes<OP>()];
    const int64_t m = blockIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const Lane ln = lane_id();
    const GlobalA<N128_NB, IN> src{static_cast<const char*>(A) + m * 128 * 128 * (IN == OP_F32 ? 4 : 2), ln};
    (void)n_mat;
    v4f Xt[9];
    Opnd<OP> yt[9];
    char* const nxt = lds + MailTiles<OP>::BYTES;
    float* const patch = reinterpret_cast<float*>(lds) + w * STORE_LDS_FLOATS;
    TRIINV_PER_WAVE(w, (neumann128_prepare<OP, W>(src, Xt, yt, lds, ln)))
    // in place: every wave has read its tiles of A before any wave stores (a barrier lies between)
    TRIINV_PER_WAVE(w, (neumann128_run<OP, W>(Xt, yt, out_matrix(T, m, 128, out_dt), lds, nxt, patch, ln)))
}

template <int KD, int OP, int DKS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(OP == OP_F32 ? 2 : 3))) void k_gdn_tri_inv_neumann128(const void* __restrict__ K, const float* __restrict__ beta,
                                                                const float* __restrict__ g, float* __restrict__ T,
                                                                uint32_t n_chunk, InvMap map, int H, int d_k, uint8_t out_dt)
{
    arguments_together(n_chunk, K, beta, g, T, map);
    constexpr int C = 128;
    typedef SharedKeys128<KD, DKS> Keys;
    typedef MailTiles<OP> Mail;
    // [keys | first mailbox buffer]; the second buffer takes the keys' place (first written after the barrier that ends
    // the keys' use), beta and g are staged, by every wave for itself, where the first buffer will be
    constexpr int CUR = Keys::BYTES > Mail::BYTES ? Keys::BYTES : Mail::BYTES;
    constexpr int LDS_BYTES = CUR + Mail::BYTES;
    static_assert(4 * 2 * C * 4 <= Mail::BYTES && 4 * STORE_LDS_FLOATS * 4 <= LDS_BYTES, "staging area and store patches fit");
    __shared__ __attribute__((aligned(16))) char lds[LDS_BYTES];
    const int64_t m = head_group_swizzle(blockIdx.x, n_chunk, H);
    const uint32_t bc = (uint32_t)m / (uint32_t)H;
    const int h = (int)((uint32_t)m - bc * (uint32_t)H);
    const ChunkPos pos = locate_chunk<C>(map, bc);
    const int64_t tok0 = pos.tok0;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const Lane ln = lane_id();
    const int64_t esz = (KD == OP_F32) ? 4 : 2;
    GateVec<N128_NB> gate;
    Keys keys;
    gate.issue(beta + tok0 * H + h, g ? g + tok0 * H + h : nullptr, H, ln, pos.valid);
    keys.load(static_cast<const char*>(K) + (tok0 * H + h) * (int64_t)d_k * esz, (int64_t)H * d_k, pos.valid, w, ln);
    gate.stage(reinterpret_cast<float*>(lds + CUR) + w * 2 * C, ln);
    keys.publish(lds, w, ln);
    __syncthreads();  // keys published, and every wave is done with its staging area
    v4f Xt[9];
    Opnd<OP> yt[9];
    float* const patch = reinterpret_cast<float*>(lds) + w * STORE_LDS_FLOATS;
    TRIINV_PER_WAVE(w, (neumann128_prepare<OP, W>(SharedA128<KD, DKS, W>{keys, gate, lds, ln}, Xt, yt, lds + CUR, ln)))
    TRIINV_PER_WAVE(w, (neumann128_run<OP, W>(Xt, yt, out_matrix(T, m, C, out_dt), lds + CUR, lds, patch, ln)))
}

}  // namespace triinv
