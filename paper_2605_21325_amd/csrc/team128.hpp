// C = 128, few matrices: eight wavefronts invert one matrix together (blocked, mixed and direct-leaf recursion), wave w from tile
// row w on, as the four of team64.hpp do at C = 64:
//   keys     wave w loads those of tile row w and leaves them in LDS for the others;
//   tiles    of A: wave w its diagonal tile, one or two of the inner blocks and two of A21 (one of a tile's rows is the wave's own);
//   leaves   wave w inverts its diagonal tile;
//   32 x 32  waves 1, 3, 5 and 7 merge the leaves' pairs;
//   64 x 64  waves 0 .. 3 form the tiles of the top block's off-diagonal part, 4 .. 7 of the bottom block's;
//   128      16 tiles of the inner product, then of the outer one: two a wave, five tile products both times;
//   store    wave w the strip of tile row w.
// Where a wavefront's part depends on w, that is a matter of LDS addresses: all eight run the same code.  Every sum is the one that the kernels of larger
// calls form (c128_invert with 16-bit operands, block_recursive with fp32 ones), in the same order: a matrix's bits do not depend on how many others its
// call has.  Bound by latency: the loads, a leaf's chain, six barriers.
// With the per-channel gate (team128_kda_tiles) wave w gates tile row w, 32 channels at a time, and the same tiles are formed from what the eight leave in LDS
// (a barrier for each 32 channels, and six more).
#pragma once
#include "team64.hpp"

namespace triinv {

template <int KD, int OP, int METHOD, int DKS> struct Team128Lds {
    static constexpr int TILE = 64 * (int)sizeof(Opnd<OP>);
    // packed tiles: leaves in both orientations, A21 [b][d], the off-diagonal parts of A's two 64 x 64 diagonal blocks [block][b][d]; of the inverse the
    // four inner off-diagonal tiles, two of them in the other orientation as well, the off-diagonal parts of its 64 x 64 blocks [block][a][c]; the
    // inner product of the last merge
    static constexpr int LEAF_N = 0, LEAF_T = 8, A21 = 16, A2 = 32, INNER = 40, TURNED = INNER + 4, W2 = TURNED + 2, PQ = W2 + 8, N_TILES = PQ + 16;
    static constexpr int KEYS = N_TILES * TILE, KEY_BYTES = 8 * DKS * 64 * 16;
    static constexpr int STRIPS = KEYS;                     // in the keys' place once all tiles of A are formed
    static constexpr int STRIP_LD = 128 + 4, STRIP_BYTES = 16 * STRIP_LD * 4;
    static constexpr int GATE = KEYS + (KEY_BYTES > 8 * STRIP_BYTES ? KEY_BYTES : 8 * STRIP_BYTES);  // beta, then g log2 e
    static constexpr int SMALL = GATE + 2 * 128 * 4;        // a wave's own: turns of a leaf
    static constexpr int SMALL_FLOATS = METHOD == M_BLOCK_DIRECT ? LEAF_STRIDE : XPOSE_FLOATS;
    static constexpr int BYTES = SMALL + 8 * SMALL_FLOATS * 4;
    static_assert(BYTES <= 160 * 1024, "a compute unit holds one team");
};

// The inner merge of waves 3 and 7 is in T orientation.
__device__ __forceinline__ bool team128_inner_t(int w) { return (w >> 1) & 1; }

// What a wavefront has of A in registers once the tiles in LDS (A21, A2) are there: its diagonal tile, and with odd w the one left of it.
template <int OP> struct Team128Tiles {
    v4f n, t;
    Opnd<OP> inner;
};

// keys_loaded(): called behind the key loads.  MERGE_T: see team128_recursion.
template <int KD, int OP, int METHOD, int DKS, bool MERGE_T, class Hook>
__device__ __forceinline__ Team128Tiles<OP> team128_tiles(char* lds, const void* Kc, int64_t row_stride, const float* bc, const float* gc, int64_t tok_stride,
                                                          int valid, int w, Lane ln, Hook keys_loaded)
{
    typedef Team128Lds<KD, OP, METHOD, DKS> LY;
    typedef typename KeyVec<KD>::type kvec;
    constexpr int KSTEP = KD == OP_F32 ? 16 : 32, PER_LANE = KD == OP_F32 ? 4 : 8;
    const int lane = 16 * ln.q + ln.n, half = w >> 2, u = w & 3;
    Opnd<OP>* const tiles = reinterpret_cast<Opnd<OP>*>(lds) + lane;
    kvec* const keys = reinterpret_cast<kvec*>(lds + LY::KEYS) + lane;  // [(tile row * DKS + k-step) * 64]
    float* const beta = reinterpret_cast<float*>(lds + LY::GATE);
    const auto tile = [&](int slot) -> Opnd<OP>& { return tiles[slot * 64]; };

    // beta and g of all 128 tokens by the first two waves, the keys of tile row w by wave w; rows beyond the last token as in GateVec and GramA
    float raw_b = 0.f, raw_g = 0.f;
    const int t = 64 * w + lane;
    if (w < 2) {
        const int tc = t < valid ? t : valid - 1;
        raw_b = bc[tc * tok_stride];
        raw_g = gc ? gc[tc * tok_stride] : 0.f;
    }
    kvec own[DKS];
    const int row = 16 * w + ln.n;
    const int64_t off = (int64_t)(row < valid ? row : valid - 1) * row_stride + PER_LANE * ln.q;
#pragma unroll
    for (int s = 0; s < DKS; ++s) own[s] = *reinterpret_cast<const kvec*>(static_cast<const char*>(Kc) + (off + KSTEP * s) * (KD == OP_F32 ? 4 : 2));
    keys_loaded();
    if (w < 2) {
        beta[t] = t < valid ? raw_b : 0.f;
        beta[128 + t] = gc ? raw_g * 1.44269504088896340736f : 0.f;
    }
    if (row >= valid) {
#pragma unroll
        for (int s = 0; s < DKS; ++s) own[s] = __builtin_bit_cast(kvec, v4u{0u, 0u, 0u, 0u});
    }
#pragma unroll
    for (int s = 0; s < DKS; ++s) keys[(w * DKS + s) * 64] = own[s];
    v4f s_own = zero4();  // symmetric but for gate and mask
#pragma unroll
    for (int k = 0; k < DKS; ++k) s_own = gram_step<KD>(own[k], own[k], s_own);
    __syncthreads();  // keys, beta and g are in LDS

    // tile (i, j) of A from its products (GateVec::apply)
    const auto gated = [&](int i, int j, bool tr, v4f s) {
        const float bn = beta[16 * i + ln.n], gn = beta[128 + 16 * (tr ? i : j) + ln.n];
        const v4f bq = *reinterpret_cast<const v4f*>(&beta[16 * i + 4 * ln.q]), gq = *reinterpret_cast<const v4f*>(&beta[128 + 16 * (tr ? j : i) + 4 * ln.q]);
        v4f a;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float wgt = (tr ? bn : bq[r]) * __builtin_amdgcn_exp2f(tr ? gn - gq[r] : gq[r] - gn);
            const bool low = i != j || (tr ? ln.n > 4 * ln.q + r : 4 * ln.q + r > ln.n);
            a[r] = low ? wgt * s[r] : 0.f;
        }
        return a;
    };
    // one of the tile's rows is this wave's
    const auto off_diagonal = [&](int i, int j, bool tr) {
        const int other = i == w ? j : i;
        v4f s = zero4();
        if ((i == w) != tr) {
#pragma unroll
            for (int k = 0; k < DKS; ++k) s = gram_step<KD>(own[k], keys[(other * DKS + k) * 64], s);
        } else {
#pragma unroll
            for (int k = 0; k < DKS; ++k) s = gram_step<KD>(keys[(other * DKS + k) * 64], own[k], s);
        }
        return pack<OP>(gated(i, j, tr, s));
    };
#pragma unroll 1
    for (int e = 0; e < 2; ++e) {  // A21: tile (4 + b, d) to wave d if b - d is 0 or 1 modulo 4, else to wave 4 + b
        const int b = half ? u : (u + e) & 3, d = half ? (u + 1 + e) & 3 : u;
        tile(LY::A21 + 4 * b + d) = off_diagonal(4 + b, d, !MERGE_T);
    }
    {  // (2,0) (3,1) (2,1) (3,0) of either block
        const int b = u & 1, d = u == 1 || u == 2;
        tile(LY::A2 + 4 * half + 2 * b + d) = off_diagonal(4 * half + 2 + b, 4 * half + d, half == 0);
    }
    Opnd<OP> inner{};
    if (w & 1) inner = off_diagonal(w, w - 1, !team128_inner_t(w));
    return {gated(w, w, false, s_own), gated(w, w, true, s_own), inner};
}

// From the leaves on.  MERGE_T: the last merge in T orientation, as block_recursive has it, else as c128_merge.  finish(strip): what is to be done with the
// result once all of it is there; strip: tile row w of it, 16 plain rows of STRIP_LD floats, anything right of the diagonal tile.
template <class LY, int OP, int METHOD, bool MERGE_T, class Finish>
__device__ __forceinline__ void team128_recursion(char* lds, const Team128Tiles<OP>& own, int aux, int w, Lane ln, Finish finish)
{
    const int lane = 16 * ln.q + ln.n, half = w >> 2, u = w & 3;
    Opnd<OP>* const tiles = reinterpret_cast<Opnd<OP>*>(lds) + lane;
    float* const small = reinterpret_cast<float*>(lds + LY::SMALL) + w * LY::SMALL_FLOATS;
    const auto strip = [&](int i) { return reinterpret_cast<float*>(lds + LY::STRIPS + i * LY::STRIP_BYTES); };
    const auto tile = [&](int slot) -> Opnd<OP>& { return tiles[slot * 64]; };
    const bool inner_t = team128_inner_t(w);
    const Opnd<OP> inner = own.inner;
    v4f XN[1], XT[1];
    const v4f LN[1] = {own.n}, LT[1] = {own.t};
    if constexpr (METHOD == M_BLOCK_DIRECT)
        leaves_forward_substitution<1>(SingleTile{LT[0]}, XN, XT, small, ln);
    else if constexpr (OP == OP_F32 && METHOD == M_MIXED)
        leaves_neumann_f32<1>(LN, LT, XN, XT, small, ln, aux);
    else if constexpr (OP == OP_F32)
        leaves_block_recursive_f32<1>(LN, LT, XN, XT, small, ln);
    else if constexpr (METHOD == M_MIXED)
        leaf_neumann<OP>(LN[0], LT[0], XN[0], XT[0], ln, aux);
    else
        leaf_block_recursive<OP>(LN[0], LT[0], XN[0], XT[0], ln);
    const Opnd<OP> leaf_t = pack<OP>(XT[0]);
    tile(LY::LEAF_N + w) = pack<OP>(XN[0]);
    tile(LY::LEAF_T + w) = leaf_t;
    __syncthreads();  // the leaves and all tiles of A are in LDS, the keys are dead

    if (half == 0)
        strip_tile<LY::STRIP_LD>(strip(w), w, w, XN[0], false, ln);
    else
        strip_tile<LY::STRIP_LD>(strip(w), w, w, XT[0], true, ln);
    if (w & 1) {
        v4f x;
        if (!inner_t) {  // -T22 (A21 T11), N orientation
            x = tn<OP>(leaf_t, negated<OP>(pack<OP>(tn<OP>(inner, tile(LY::LEAF_N + w - 1), zero4()))), zero4());
            strip_tile<LY::STRIP_LD>(strip(w), w, w - 1, x, false, ln);
        } else {         // its transpose, -T11^T (A21^T T22^T)
            x = tn<OP>(tile(LY::LEAF_N + w - 1), negated<OP>(pack<OP>(tn<OP>(inner, leaf_t, zero4()))), zero4());
            strip_tile<LY::STRIP_LD>(strip(w), w, w - 1, x, true, ln);
        }
        tile(LY::INNER + (w >> 1)) = pack<OP>(x);
        if (w == 3 || w == 5) tile(LY::TURNED + (w == 5)) = pack<OP>(transpose_tile(x, small, ln));
    }
    __syncthreads();  // the 32 x 32 blocks are complete

    // acc + the sum over k in [lo, hi] of x(k)^T y(k)
    const auto sum = [&](int lo, int hi, int n, auto x, auto y) {
        v4f acc = zero4();
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (k < n && k >= lo && k <= hi) acc = tn<OP>(tile(x(k)), tile(y(k)), acc);
        return acc;
    };
    {  // tile (2 + a, c) of a 64 x 64 block
        const int a = u >> 1, c = u & 1, base = 4 * half, a2 = LY::A2 + 4 * half, in = LY::INNER + 2 * half;
        const auto t11 = [&](int d, int k) { return d == k ? LY::LEAF_N + base + d : in; };
        const auto t22 = [&](int i, int k) { return i == k ? LY::LEAF_T + base + 2 + i : in + 1; };
        v4f x = zero4();
        if (half == 0) {  // -T22 (A21 T11), N orientation
#pragma unroll
            for (int b = 0; b < 2; ++b)
                if (b <= a) {
                    const v4f p = sum(c, 1, 2, [&](int d) { return a2 + 2 * b + d; }, [&](int d) { return t11(d, c); });
                    x = tn<OP>(tile(t22(a, b)), negated<OP>(pack<OP>(p)), x);
                }
        } else {          // its transpose
#pragma unroll
            for (int d = 0; d < 2; ++d)
                if (d >= c) {
                    const v4f q = sum(0, a, 2, [&](int b) { return a2 + 2 * b + d; }, [&](int b) { return t22(a, b); });
                    x = tn<OP>(tile(t11(d, c)), negated<OP>(pack<OP>(q)), x);
                }
        }
        tile(LY::W2 + 4 * half + 2 * a + c) = pack<OP>(x);
        if (half == 0)
            strip_tile<LY::STRIP_LD>(strip(2 + a), 2 + a, c, x, false, ln);
        else
            strip_tile<LY::STRIP_LD>(strip(6 + a), 6 + a, 4 + c, x, true, ln);
    }
    __syncthreads();  // the 64 x 64 blocks are complete

    // tiles of T11 in N orientation and of T22 in T orientation
    const auto t11 = [&](int d, int c) { return d == c ? LY::LEAF_N + d : d == 1 ? LY::INNER : d == 3 && c == 2 ? LY::TURNED : LY::W2 + 2 * (d - 2) + c; };
    const auto t22 = [&](int a, int b) { return a == b ? LY::LEAF_T + 4 + a : a == 1 ? LY::TURNED + 1 : a == 3 && b == 2 ? LY::INNER + 3 : LY::W2 + 4 + 2 * (a - 2) + b; };
    const int one = w >> 1;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int two = e == 0 ? w & 1 : 3 - (w & 1);
        if (MERGE_T) {  // Q(a, d) = -sum over b <= a of A(b, d)^T T22(a, b)^T
            const int d = one, a = two;
            tile(LY::PQ + 4 * a + d) = negated<OP>(pack<OP>(sum(0, a, 4, [&](int b) { return LY::A21 + 4 * b + d; }, [&](int b) { return t22(a, b); })));
        } else {        // P(b, c) = -sum over d >= c of A(b, d) T11(d, c)
            const int b = one, c = two;
            tile(LY::PQ + 4 * b + c) = negated<OP>(pack<OP>(sum(c, 3, 4, [&](int d) { return LY::A21 + 4 * b + d; }, [&](int d) { return t11(d, c); })));
        }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int two = e == 0 ? w & 1 : 3 - (w & 1);
        if (MERGE_T) {
            const int a = one, c = two;
            const v4f x = sum(c, 3, 4, [&](int d) { return t11(d, c); }, [&](int d) { return LY::PQ + 4 * a + d; });
            strip_tile<LY::STRIP_LD>(strip(4 + a), 4 + a, c, x, true, ln);
        } else {
            const int c = one, a = two;
            const v4f x = sum(0, a, 4, [&](int b) { return t22(a, b); }, [&](int b) { return LY::PQ + 4 * b + c; });
            strip_tile<LY::STRIP_LD>(strip(4 + a), 4 + a, c, x, false, ln);
        }
    }
    __syncthreads();  // the strips are complete
    finish(strip(w));
}

template <int KD, int OP, int METHOD, int DKS>
__global__ __launch_bounds__(512) void k_gdn_tri_inv_team128(const void* __restrict__ K, const float* __restrict__ beta, const float* __restrict__ g,
                                                             float* __restrict__ T, uint32_t n_chunk, InvMap map, int H, int d_k, uint8_t aux, uint8_t out_dt)
{
    arguments_together(n_chunk, K, beta, g, T, map);
    __shared__ __attribute__((aligned(16))) char lds[Team128Lds<KD, OP, METHOD, DKS>::BYTES];
    const uint32_t m = blockIdx.x, bc = m / (uint32_t)H;
    const int h = (int)(m - bc * (uint32_t)H);
    const ChunkPos pos = locate_chunk<128>(map, bc);
    const int64_t tok0 = pos.tok0;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const void* const Kc = static_cast<const char*>(K) + (tok0 * H + h) * (int64_t)d_k * (KD == OP_F32 ? 4 : 2);
    const Lane ln = lane_id();
    const Out Tm = out_matrix(T, m, 128, out_dt);
    const auto own = team128_tiles<KD, OP, METHOD, DKS, OP == OP_F32>(lds, Kc, (int64_t)H * d_k, beta + tok0 * H + h, g ? g + tok0 * H + h : nullptr, H,
                                                                      pos.valid, w, ln, NoHook());
    team128_recursion<Team128Lds<KD, OP, METHOD, DKS>, OP, METHOD, OP == OP_F32>(
        lds, own, aux, w, ln, [&](float* strip) { flush_strip<8, false, 128 + 4>(Tm, w, strip, ln); });
}

// Per-channel gate, d_k any multiple of 32: the factors of c128_kda_gram, by the wave whose keys and gates they are made of, 32 channels at a time through
// LDS in place of what the recursion keeps there, in two buffers.
template <int OP, int METHOD> struct Team128KdaLds : Team128Lds<OP_F16, OP, METHOD, 0> {
    typedef Team128Lds<OP_F16, OP, METHOD, 0> BASE;
    // of one k-step: every wave's factor for A21; left factors of tile rows 2, 3 of either block; right factors of (1,0) (3,0) (2,1) (3,2) of either
    static constexpr int MINE = 0, LEFT = 8, RIGHT = 12, SLOTS = 20;
    static constexpr int GATES = BASE::GATE - 8 * 1536;  // per wave: anchors [tile row][32 channels], channel factors [q][4][8]
    static_assert(2 * SLOTS * 64 * (int)sizeof(GOp<OP>) <= GATES, "no overlap");
};

template <int OP, int METHOD, bool K16>
__device__ __forceinline__ Team128Tiles<OP> team128_kda_tiles(char* lds, const void* Kc, bool is_f16, const float* gc, int64_t row_stride, int d_k,
                                                              const float* bc, int64_t tok_stride, int valid, int w, Lane ln)
{
    typedef Team128KdaLds<OP, METHOD> LY;
    constexpr float LOG2E = 1.44269504088896340736f;
    constexpr int AHEAD = 4;  // k-steps in flight: all of d_k = 128
    const int lane = 16 * ln.q + ln.n, half = w >> 2, u = w & 3;
    GOp<OP>* const xchg = reinterpret_cast<GOp<OP>*>(lds) + lane;
    float* const beta = reinterpret_cast<float*>(lds + LY::GATE);
    float* const anc = reinterpret_cast<float*>(lds + LY::GATES) + w * 384;
    float* const fac = anc + 256 + ln.q * 32;

    const int t = 64 * w + lane;
    float raw_b = 0.f;
    if (w < 2) raw_b = t < valid ? bc[t * tok_stride] : 0.f;
    const int n_step = d_k / 32;
    const int row = 16 * w + ln.n, arow = 16 * (lane >> 3);
    const int64_t off = (int64_t)(row < valid ? row : valid - 1) * row_stride + 8 * ln.q;
    const int64_t aoff = (int64_t)(arow < valid ? arow : valid - 1) * row_stride + 4 * (lane & 7);
    RawKey8<K16> key[AHEAD];
    v4f G[AHEAD][2], A[AHEAD];
    const auto request = [&](int i, int s) {
        if (s >= n_step) return;
        A[i] = *reinterpret_cast<const v4f*>(gc + aoff + 32 * s);
        G[i][0] = *reinterpret_cast<const v4f*>(gc + off + 32 * s);
        G[i][1] = *reinterpret_cast<const v4f*>(gc + off + 32 * s + 4);
        key[i] = load_key8<K16>(Kc, off + 32 * s);
    };
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) request(i, i);
    if (w < 2) beta[t] = raw_b;

    v4f own_n = zero4(), own_t = zero4(), a_inner = zero4(), a2 = zero4(), a21[2] = {zero4(), zero4()};
    for (int s0 = 0; s0 < n_step; s0 += AHEAD) {
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
            const int s = s0 + i;
            if (s >= n_step) break;
            *reinterpret_cast<v4f*>(&anc[4 * lane]) = A[i];
            wave_lds_sync();
            // channel factors: of A21 (anchors of this tile row and the chunk's row 64), then of tiles (u + 1 .. 3, u)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int e = ln.n + 16 * k, p = e >> 3, c = 8 * ln.q + (e & 7);
                const int below = 4 * half + (u + p < 4 ? u + p : 3);
                const int hi = p ? below : half ? w : 4, lo = p ? w : half ? 4 : w;
                fac[e] = __builtin_amdgcn_exp2f((anc[32 * hi + c] - anc[32 * lo + c]) * LOG2E);
            }
            wave_lds_sync();
            if (row >= valid) key[i] = RawKey8<K16>{};
            float kv[8], left[8], diag[8], m[8];
            widen_key8<K16>(key[i], is_f16, kv);
            const auto factor = [&](int p, int r) { return fac[8 * p + r]; };
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const float e = (G[i][r / 4][r % 4] - anc[32 * w + 8 * ln.q + r]) * LOG2E;
                left[r] = kv[r] * __builtin_amdgcn_exp2f(e);
                diag[r] = kv[r] * __builtin_amdgcn_exp2f(-e);
                m[r] = (half ? left[r] : diag[r]) * factor(0, r);
            }
            const auto right = [&](int p) {
                float x[8];
#pragma unroll
                for (int r = 0; r < 8; ++r) x[r] = diag[r] * factor(p, r);
                return gpack<OP>(x);
            };
            const GOp<OP> p_left = gpack<OP>(left), p_diag = gpack<OP>(diag), mine = gpack<OP>(m), p_right2 = right(2);
            GOp<OP>* const x = xchg + (s & 1) * LY::SLOTS * 64;
            x[(LY::MINE + w) * 64] = mine;
            if (u >= 2) x[(LY::LEFT + 2 * half + u - 2) * 64] = p_left;
            if (u < 3) x[(LY::RIGHT + 4 * half + (u == 0 ? 0 : u + 1)) * 64] = right(1);
            if (u == 0) x[(LY::RIGHT + 4 * half + 1) * 64] = right(3);
            __syncthreads();  // this k-step's factors are in LDS (nobody reads the buffer of the step before last any more)
            if (METHOD != M_BLOCK_DIRECT) own_n = gstep<OP>(p_left, p_diag, own_n);
            own_t = gstep<OP>(p_diag, p_left, own_t);
            // tile (i, j) from its left and right factor
            const auto product = [&](bool tr, const GOp<OP>& l, const GOp<OP>& r, v4f& acc) {
                if (tr)
                    acc = gstep<OP>(r, l, acc);
                else
                    acc = gstep<OP>(l, r, acc);
            };
            if (w & 1) product(!team128_inner_t(w), p_left, x[(LY::RIGHT + 4 * half + (u == 1 ? 0 : 3)) * 64], a_inner);
            if (u < 2)
                product(half == 0, x[(LY::LEFT + 2 * half + u) * 64], p_right2, a2);
            else
                product(half == 0, p_left, x[(LY::RIGHT + 4 * half + (u == 2 ? 2 : 1)) * 64], a2);
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                if (half == 0)
                    a21[e] = gstep<OP>(mine, x[(LY::MINE + 4 + ((u + e) & 3)) * 64], a21[e]);
                else
                    a21[e] = gstep<OP>(x[(LY::MINE + ((u + 1 + e) & 3)) * 64], mine, a21[e]);
            }
            request(i, s + AHEAD);
        }
    }
    __syncthreads();  // the last factors have been read

    Opnd<OP>* const tiles = reinterpret_cast<Opnd<OP>*>(lds) + lane;
    const auto scaled = [&](int i, bool tr, v4f s) {  // by beta of the row
        const float bn = beta[16 * i + ln.n];
        const v4f bq = *reinterpret_cast<const v4f*>(&beta[16 * i + 4 * ln.q]);
        v4f a;
#pragma unroll
        for (int r = 0; r < 4; ++r) a[r] = (tr ? bn : bq[r]) * s[r];
        return a;
    };
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int b = half ? u : (u + e) & 3, d = half ? (u + 1 + e) & 3 : u;
        tiles[(LY::A21 + 4 * b + d) * 64] = pack<OP>(scaled(4 + b, true, a21[e]));
    }
    {
        const int b = u & 1, d = u == 1 || u == 2;
        tiles[(LY::A2 + 4 * half + 2 * b + d) * 64] = pack<OP>(scaled(4 * half + 2 + b, half == 0, a2));
    }
    own_n = scaled(w, false, own_n);
    own_t = scaled(w, true, own_t);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        own_n[r] = 4 * ln.q + r > ln.n ? own_n[r] : 0.f;
        own_t[r] = ln.n > 4 * ln.q + r ? own_t[r] : 0.f;
    }
    return {own_n, own_t, pack<OP>(scaled(w, !team128_inner_t(w), a_inner))};
}

template <int OP, int METHOD, bool K16>
__global__ __launch_bounds__(512) void k_kda_tri_inv_team128(const void* __restrict__ K, const float* __restrict__ beta, const float* __restrict__ g,
                                                             float* __restrict__ T, uint32_t n_chunk, InvMap map, int H, int d_k, uint8_t k_dt, uint8_t aux,
                                                             uint8_t out_dt)
{
    arguments_together(n_chunk, K, beta, g, T, map);
    typedef Team128KdaLds<OP, METHOD> LY;
    __shared__ __attribute__((aligned(16))) char lds[LY::BYTES];
    const uint32_t m = blockIdx.x, bc = m / (uint32_t)H;
    const int h = (int)(m - bc * (uint32_t)H);
    const ChunkPos pos = locate_chunk<128>(map, bc);
    const int64_t tok0 = pos.tok0, e0 = (tok0 * H + h) * (int64_t)d_k;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const Lane ln = lane_id();
    const Out Tm = out_matrix(T, m, 128, out_dt);
    const auto own = team128_kda_tiles<OP, METHOD, K16>(lds, static_cast<const char*>(K) + e0 * (K16 ? 2 : 4), k_dt == OP_F16, g + e0, (int64_t)H * d_k, d_k,
                                                        beta + tok0 * H + h, H, pos.valid, w, ln);
    team128_recursion<LY, OP, METHOD, false>(lds, own, aux, w, ln, [&](float* strip) { flush_strip<8, false, 128 + 4>(Tm, w, strip, ln); });
}

}  // namespace triinv
