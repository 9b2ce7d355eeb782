// C = 64, few matrices: four wavefronts invert one matrix together, through the recursion and the store too (blocked, mixed and direct-leaf
// recursion).  One wavefront alone takes its matrix instructions and its strips one after the other; here each of the four SIMDs of a
// compute unit has a share:
//   leaves  wave w inverts diagonal tile w;
//   32 x 32 waves 1 and 3 merge leaves (0, 1) and (2, 3);
//   64 x 64 wave 2 a + c forms tile (2 + a, c) of the off-diagonal block;
//   store   wave w the strip of tile row w.
// Every sum is the one that a wavefront alone forms (block_recursive), in the same order: a matrix's bits do not depend on how many others its
// call has.  Bound by latency: the loads, a leaf's chain, four barriers.
#pragma once
#include "kernels.hpp"

namespace triinv {

template <int METHOD> constexpr bool team64_method() { return METHOD == M_BLOCK || METHOD == M_MIXED || METHOD == M_BLOCK_DIRECT; }

// LDS from the leaves on: packed tiles [tile][lane] (leaves in both orientations, A21, the two inner off-diagonal tiles), the strips of the result,
// and a little of every wave's own (gate staging, turns of a leaf).
template <int OP, int METHOD> struct Team64Lds {
    static constexpr int LEAF_N = 0, LEAF_T = 4, A21 = 8, INNER = 12, N_TILES = 14;
    static constexpr int STRIPS = N_TILES * 64 * (int)sizeof(Opnd<OP>);
    static constexpr int STRIP_LD = 16 * 4 + 4, STRIP_BYTES = 16 * STRIP_LD * 4;
    static constexpr int SMALL = STRIPS + 4 * STRIP_BYTES;
    static constexpr int SMALL_FLOATS = METHOD == M_BLOCK_DIRECT ? LEAF_STRIDE : XPOSE_FLOATS;
    static constexpr int BYTES = SMALL + 4 * SMALL_FLOATS * 4;
    static_assert(SMALL_FLOATS >= gate_lds_floats<4>() && STRIPS % 16 == 0, "the gate is staged there");
    static __device__ __forceinline__ float* small(char* area, int w) { return reinterpret_cast<float*>(area + SMALL) + w * SMALL_FLOATS; }
};

// One tile as a source of its own.
struct SingleTile {
    v4f t;
    template <bool> __device__ __forceinline__ v4f get(int, int) const { return t; }
};

// Wave W's part, from its diagonal tile of A (both orientations; the direct leaves use LT alone) and off_diagonal(i, j, T orientation?), which gives the
// tiles of A below the diagonal: (2,0) (3,0) to wave 0, (1,0) (3,1) to wave 1, (2,1) to wave 2, (3,2) to wave 3.
// finish(strip): what is to be done with the result once all of it is there; strip: tile row W of it, 16 plain rows of STRIP_LD floats, unit diagonal and zeros
// above it in the diagonal tile, anything right of that.
template <int OP, int METHOD, int W, class OffDiagonal, class Finish>
__device__ __forceinline__ void team64_recursion(char* area, v4f diag_n, v4f diag_t, OffDiagonal off_diagonal, int aux, Lane ln, Finish finish)
{
    typedef Team64Lds<OP, METHOD> LY;
    Opnd<OP>* const tiles = reinterpret_cast<Opnd<OP>*>(area) + 16 * ln.q + ln.n;
    const auto strip = [&](int i) { return reinterpret_cast<float*>(area + LY::STRIPS + i * LY::STRIP_BYTES); };
    const auto share_a21 = [&](int b, int d) { tiles[(LY::A21 + 2 * b + d) * 64] = pack<OP>(off_diagonal(2 + b, d, false)); };
    Opnd<OP> inner{};  // A of this wave's inner merge
    if (W == 0) {
        share_a21(0, 0);
        share_a21(1, 0);
    } else if (W == 1) {
        inner = pack<OP>(off_diagonal(1, 0, true));
        share_a21(1, 1);
    } else if (W == 2) {
        share_a21(0, 1);
    } else {
        inner = pack<OP>(off_diagonal(3, 2, false));
    }
    v4f XN[1], XT[1];
    const v4f LN[1] = {diag_n}, LT[1] = {diag_t};
    float* const small = LY::small(area, W);
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
    const Opnd<OP> leaf_n = pack<OP>(XN[0]), leaf_t = pack<OP>(XT[0]);
    tiles[(LY::LEAF_N + W) * 64] = leaf_n;
    tiles[(LY::LEAF_T + W) * 64] = leaf_t;
    strip_tile<LY::STRIP_LD>(strip(W), W, W, W < 2 ? XN[0] : XT[0], W >= 2, ln);
    __syncthreads();  // the leaves and A21 are in LDS

    if (W == 1) {  // -T22 (A21 T11), N orientation
        const v4f t = tn<OP>(leaf_t, negated<OP>(pack<OP>(tn<OP>(inner, tiles[(LY::LEAF_N + 0) * 64], zero4()))), zero4());
        tiles[(LY::INNER + 0) * 64] = pack<OP>(t);
        strip_tile<LY::STRIP_LD>(strip(1), 1, 0, t, false, ln);
    } else if (W == 3) {  // its transpose, -T11^T (A21^T T22^T)
        const v4f t = tn<OP>(tiles[(LY::LEAF_N + 2) * 64], negated<OP>(pack<OP>(tn<OP>(inner, leaf_t, zero4()))), zero4());
        tiles[(LY::INNER + 1) * 64] = pack<OP>(t);
        strip_tile<LY::STRIP_LD>(strip(3), 3, 2, t, true, ln);
    }
    __syncthreads();  // the two 32 x 32 blocks are complete

    // tile (2 + a, c) of -T22 A21 T11, T orientation
    constexpr int a = W / 2, c = W % 2;
    Opnd<OP> t22[2] = {tiles[(a == 0 ? LY::LEAF_T + 2 : LY::INNER + 1) * 64], tiles[(LY::LEAF_T + 3) * 64]}, Q[2];
#pragma unroll
    for (int d = c; d < 2; ++d) {
        v4f acc = zero4();
#pragma unroll
        for (int b = 0; b <= a; ++b) acc = tn<OP>(tiles[(LY::A21 + 2 * b + d) * 64], t22[b], acc);
        Q[d] = negated<OP>(pack<OP>(acc));
    }
    v4f t = zero4();
#pragma unroll
    for (int d = c; d < 2; ++d) t = tn<OP>(tiles[(d == c ? LY::LEAF_N + d : LY::INNER + 0) * 64], Q[d], t);
    strip_tile<LY::STRIP_LD>(strip(2 + a), 2 + a, c, t, true, ln);
    __syncthreads();  // the strips are complete
    finish(strip(W));
}

// The result stored: wave W tile row W.
template <int W> struct Team64Store {
    Out Tm;
    Lane ln;
    __device__ __forceinline__ void operator()(float* strip) const { flush_strip<4, false, 16 * 4 + 4>(Tm, W, strip, ln); }
};

// Scalar / no-gate kinds, d_k = 64 or 128, fp32 operands (304 fp32 matrix instructions of 32 cycles for 64 fp32 channels): wave w loads the keys of tile row w,
// leaves them in LDS for the others and forms its tiles of A.
// keys_loaded(): called behind the key loads.
template <int KD, int OP, int METHOD, int DKS, int W, class Hook, class Finish>
__device__ __forceinline__ void team64_invert(char* key_lds, char* area, const void* Kc, int64_t row_stride, const float* bc, const float* gc,
                                              int64_t tok_stride, int valid, int aux, Lane ln, Hook keys_loaded, Finish finish)
{
    typedef typename KeyVec<KD>::type kvec;
    constexpr int KSTEP = KD == OP_F32 ? 16 : 32, PER_LANE = KD == OP_F32 ? 4 : 8;
    kvec* const keys = reinterpret_cast<kvec*>(key_lds) + 16 * ln.q + ln.n;  // [(tile row * DKS + k-step) * 64]
    GateVec<4> gate;
    gate.issue(bc, gc, tok_stride, ln, valid);
    kvec own[DKS];
    const int row = 16 * W + ln.n;
    const int64_t off = (int64_t)(row < valid ? row : valid - 1) * row_stride + PER_LANE * ln.q;
#pragma unroll
    for (int s = 0; s < DKS; ++s) own[s] = *reinterpret_cast<const kvec*>(static_cast<const char*>(Kc) + (off + KSTEP * s) * (KD == OP_F32 ? 4 : 2));
    keys_loaded();
    if (row >= valid) {
#pragma unroll
        for (int s = 0; s < DKS; ++s) own[s] = __builtin_bit_cast(kvec, v4u{0u, 0u, 0u, 0u});
    }
    gate.stage(Team64Lds<OP, METHOD>::small(area, W), ln);
#pragma unroll
    for (int s = 0; s < DKS; ++s) keys[(W * DKS + s) * 64] = own[s];
    v4f s_own = zero4();  // symmetric but for gate and mask
#pragma unroll
    for (int t = 0; t < DKS; ++t) s_own = gram_step<KD>(own[t], own[t], s_own);
    __syncthreads();  // the keys are in LDS
    // one of the tile's rows is this wave's
    const auto off_diagonal = [&](int i, int j, bool tr) {
        const int other = i == W ? j : i;
        v4f s = zero4();
#pragma unroll
        for (int t = 0; t < DKS; ++t) {
            const kvec k = keys[(other * DKS + t) * 64];
            s = (i == W) != tr ? gram_step<KD>(own[t], k, s) : gram_step<KD>(k, own[t], s);
        }
        return tr ? gate.template apply<true>(i, j, s, ln) : gate.template apply<false>(i, j, s, ln);
    };
    team64_recursion<OP, METHOD, W>(area, gate.template apply<false>(W, W, s_own, ln), gate.template apply<true>(W, W, s_own, ln), off_diagonal, aux, ln, finish);
}

template <int KD, int OP, int METHOD, int DKS>
__global__ __launch_bounds__(256) void k_gdn_tri_inv_team64(const void* __restrict__ K, const float* __restrict__ beta, const float* __restrict__ g,
                                                            float* __restrict__ T, uint32_t n_chunk, InvMap map, int H, int d_k, uint8_t aux, uint8_t out_dt)
{
    arguments_together(n_chunk, K, beta, g, T, map);
    __shared__ __attribute__((aligned(16))) char key_lds[4 * DKS * 64 * 16];
    __shared__ __attribute__((aligned(16))) char area[Team64Lds<OP, METHOD>::BYTES];
    const uint32_t m = blockIdx.x, bc = m / (uint32_t)H;
    const int h = (int)(m - bc * (uint32_t)H);
    const ChunkPos pos = locate_chunk<64>(map, bc);
    const int64_t tok0 = pos.tok0;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const Lane ln = lane_id();
    const void* const Kc = static_cast<const char*>(K) + (tok0 * H + h) * (int64_t)d_k * (KD == OP_F32 ? 4 : 2);
    const Out Tm = out_matrix(T, m, 64, out_dt);
    TRIINV_PER_WAVE(w, (team64_invert<KD, OP, METHOD, DKS, W>(key_lds, area, Kc, (int64_t)H * d_k, beta + tok0 * H + h, g ? g + tok0 * H + h : nullptr, H,
                                                              pos.valid, aux, ln, NoHook(), Team64Store<W>{Tm, ln})))
}

// A formed in a channel loop (team_gram_products): the products stay where they are, what the loop needed beside them makes room for the rest.
template <int OPG, int OP, int METHOD, bool GATED> struct Team64Loop {
    static constexpr int AREA = GramProducts<4, METHOD, GATED>::COUNT * TeamLds<OPG, 4, GATED>::PLANE;
    static constexpr int LOOP = team_lds_bytes<OPG, 4, METHOD, GATED>();
    static constexpr int BYTES = AREA + Team64Lds<OP, METHOD>::BYTES > LOOP ? AREA + Team64Lds<OP, METHOD>::BYTES : LOOP;
};

// Per-channel gate.
template <int OP, int METHOD, int W, class Finish>
__device__ __forceinline__ void team64_from_channels(const Team& team, const float* bc, int64_t tok_stride, int valid, int aux, Lane ln, Finish finish)
{
    typedef GramProducts<4, METHOD, true> Products;
    char* const area = team.lds + Team64Loop<OP, OP, METHOD, true>::AREA;
    float* const beta = Team64Lds<OP, METHOD>::small(area, W);
    const int l = 16 * ln.q + ln.n;
    beta[l] = l < valid ? bc[l * tok_stride] : 0.f;
    wave_lds_sync();
    v4f beta_n, beta_q[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        beta_n[i] = beta[16 * i + ln.n];
        beta_q[i] = *reinterpret_cast<const v4f*>(&beta[16 * i + 4 * ln.q]);
    }
    wave_lds_sync();
    // beta_i row scaling and the strictly-lower mask
    const auto tile = [&](int k, int i, int j, bool tr) {
        v4f a = team_product<OP, 4, true>(team, k, ln);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const bool low = i != j || (tr ? ln.n > 4 * ln.q + r : 4 * ln.q + r > ln.n);
            a[r] = low ? (tr ? beta_n[i] : beta_q[i][r]) * a[r] : 0.f;
        }
        return a;
    };
    const v4f diag_t = tile(Products::find(W, W, true), W, W, true);
    const v4f diag_n = METHOD == M_BLOCK_DIRECT ? zero4() : tile(Products::find(W, W, false), W, W, false);
    team64_recursion<OP, METHOD, W>(area, diag_n, diag_t, [&](int i, int j, bool tr) { return tile(Products::find(i, j, tr), i, j, tr); }, aux, ln, finish);
}

template <int OP, int METHOD>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_kda_tri_inv_team64(const void* __restrict__ K, const float* __restrict__ beta,
                                                            const float* __restrict__ g, float* __restrict__ T, uint32_t n_chunk, InvMap map, int H, int d_k,
                                                            uint8_t k_dt, uint8_t aux, uint8_t out_dt)
{
    arguments_together(n_chunk, K, beta, g, T, map);
    __shared__ __attribute__((aligned(16))) char lds[Team64Loop<OP, OP, METHOD, true>::BYTES];
    const uint32_t m = blockIdx.x, bc = m / (uint32_t)H;
    const int h = (int)(m - bc * (uint32_t)H);
    const ChunkPos pos = locate_chunk<64>(map, bc);
    const int64_t tok0 = pos.tok0, e0 = (tok0 * H + h) * (int64_t)d_k, row_stride = (int64_t)H * d_k;
    const Lane ln = lane_id();
    const void* const Kc = static_cast<const char*>(K) + e0 * (k_dt == OP_F32 ? 4 : 2);
    const Team team = this_team(lds);
    if (k_dt == OP_F32)
        team_gram_products<OP, 4, METHOD, false, true>(Kc, false, g + e0, row_stride, d_k / 32, ln, pos.valid, team);
    else
        team_gram_products<OP, 4, METHOD, true, true>(Kc, k_dt == OP_F16, g + e0, row_stride, d_k / 32, ln, pos.valid, team);
    const Out Tm = out_matrix(T, m, 64, out_dt);
    TRIINV_PER_WAVE(team.w, (team64_from_channels<OP, METHOD, W>(team, beta + tok0 * H + h, H, pos.valid, aux, ln, Team64Store<W>{Tm, ln})))
}

// Scalar / no-gate kinds, any d_k.
template <int KD, int OP, int METHOD, int W, class Finish>
__device__ __forceinline__ void team64_from_products(const Team& team, const float* bc, const float* gc, int64_t tok_stride, int valid, int aux, Lane ln, Finish finish)
{
    typedef GramProducts<4, METHOD, false> Products;
    char* const area = team.lds + Team64Loop<KD, OP, METHOD, false>::AREA;
    GateVec<4> gate;
    gate.load(bc, gc, tok_stride, Team64Lds<OP, METHOD>::small(area, W), ln, valid);
    const auto tile = [&](int k, int i, int j, bool tr) {
        const v4f s = team_product<KD, 4, false>(team, k, ln);
        return tr ? gate.template apply<true>(i, j, s, ln) : gate.template apply<false>(i, j, s, ln);
    };
    constexpr int own = Products::find(W, W, true);
    team64_recursion<OP, METHOD, W>(area, tile(own, W, W, false), tile(own, W, W, true), [&](int i, int j, bool tr) { return tile(Products::find(i, j, tr), i, j, tr); },
                                    aux, ln, finish);
}

template <int KD, int OP, int METHOD>
__global__ __launch_bounds__(256) void k_gdn_any_dk_tri_inv_team64(const void* __restrict__ K, const float* __restrict__ beta, const float* __restrict__ g,
                                                            float* __restrict__ T, uint32_t n_chunk, InvMap map, int H, int d_k, uint8_t aux, uint8_t out_dt)
{
    arguments_together(n_chunk, K, beta, g, T, map);
    __shared__ __attribute__((aligned(16))) char lds[Team64Loop<KD, OP, METHOD, false>::BYTES];
    const uint32_t m = blockIdx.x, bc = m / (uint32_t)H;
    const int h = (int)(m - bc * (uint32_t)H);
    const ChunkPos pos = locate_chunk<64>(map, bc);
    const int64_t tok0 = pos.tok0, row_stride = (int64_t)H * d_k;
    const Lane ln = lane_id();
    const void* const Kc = static_cast<const char*>(K) + (tok0 * H + h) * (int64_t)d_k * (KD == OP_F32 ? 4 : 2);
    const Team team = this_team(lds);
    team_gram_products<KD, 4, METHOD, KD != OP_F32, false>(Kc, KD == OP_F16, nullptr, row_stride, d_k / 32, ln, pos.valid, team);
    const Out Tm = out_matrix(T, m, 64, out_dt);
    TRIINV_PER_WAVE(team.w, (team64_from_products<KD, OP, METHOD, W>(team, beta + tok0 * H + h, g ? g + tok0 * H + h : nullptr, H, pos.valid, aux, ln,
                                                                         Team64Store<W>{Tm, ln})))
}

}  // namespace triinv
