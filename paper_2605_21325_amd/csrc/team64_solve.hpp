// The teams of team64.hpp with the inverse applied instead of stored (W_k = T diag(s_k) X_k, blocked and mixed recursion): wave w forms tile row w of W,
// from its strip of T and tile rows 0 .. w of X, which it requested ahead of the recursion.
#pragma once
#include "solve.hpp"
#include "team64.hpp"

namespace triinv {

// One chunk's right-hand sides for wave W: the loads of the first one start with `issue`, the rest is done as the recursion's last step.
template <int OP, int W, int NRHS> struct Team64Apply {
    static constexpr int VEC = RhsX<OP, 4>::VEC, LD = 16 * 4 + 4;
    const RhsList& rhs;
    int64_t tok0;
    int h, H, valid;
    Lane ln;
    RhsX<OP, 4> x;

    __device__ __forceinline__ Team64Apply(const RhsList& rhs_, int64_t tok0_, int h_, int H_, int valid_, Lane ln_)
        : rhs(rhs_), tok0(tok0_), h(h_), H(H_), valid(valid_), ln(ln_)
    {
    }
    __device__ __forceinline__ void issue(int k)
    {
        x.init(rhs.r[k], tok0, h, H, valid, ln);
        x.issue(0, 0, W + 1);
    }
    __device__ __forceinline__ void operator()(const float* strip)
    {
        v4f T[W + 1];  // T orientation
#pragma unroll
        for (int j = 0; j <= W; ++j) T[j] = *reinterpret_cast<const v4f*>(&strip[ln.n * LD + 16 * j + 4 * ln.q]);
#pragma unroll
        for (int k = 0; k < NRHS; ++k) {
            if (k > 0) issue(k);
            Opnd<OP> Top[W + 1];  // columns scaled by s in fp32, then rounded to the operand type
#pragma unroll
            for (int j = 0; j <= W; ++j) Top[j] = pack<OP>(T[j] * x.s_q[j]);
            const int n_group = x.n_group();
#pragma unroll 1
            for (int gi = 0;;) {
                v4f acc[VEC];
#pragma unroll
                for (int c = 0; c < VEC; ++c) acc[c] = zero4();
#pragma unroll
                for (int j = 0; j <= W; ++j)
#pragma unroll
                    for (int c = 0; c < VEC; ++c) acc[c] = tn<OP>(Top[j], x_operand<OP>(x.raw[j], c), acc[c]);
                const int done = gi++;
                if (gi < n_group) x.issue(gi, 0, W + 1);
                x.store(done, W, acc);
                if (gi >= n_group) break;
            }
        }
    }
};

// Scalar / no-gate kinds, d_k = 64 or 128.
template <int KD, int OP, int METHOD, int DKS, int NRHS, int W>
__device__ __forceinline__ void team64_solve(char* key_lds, char* area, const void* Kc, int64_t row_stride, const float* bc, const float* gc, const RhsList& rhs,
                                             int64_t tok0, int h, int H, int valid, int aux, Lane ln)
{
    Team64Apply<OP, W, NRHS> apply(rhs, tok0, h, H, valid, ln);
    team64_invert<KD, OP, METHOD, DKS, W>(key_lds, area, Kc, row_stride, bc, gc, H, valid, aux, ln, [&]() { apply.issue(0); },
                                          [&](float* strip) { apply(strip); });
}

template <int KD, int OP, int METHOD, int DKS, int NRHS>
__global__ __launch_bounds__(256) void k_gdn_tri_solve_team64(const void* __restrict__ K, const float* __restrict__ beta, const float* __restrict__ g, RhsList rhs,
                                                              int64_t n_chunk, SolveMap<NRHS == 1> map, int H, int d_k, int aux)
{
    arguments_together(n_chunk, K, beta, g, rhs.r[0].X, map);
    __shared__ __attribute__((aligned(16))) char key_lds[4 * DKS * 64 * 16];
    __shared__ __attribute__((aligned(16))) char area[Team64Lds<OP, METHOD>::BYTES];
    const uint32_t m = blockIdx.x, bc = m / (uint32_t)H;
    const int h = (int)(m - bc * (uint32_t)H);
    const ChunkPos pos = locate_chunk<64>(map, bc);
    const int64_t tok0 = pos.tok0;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const Lane ln = lane_id();
    const void* const Kc = static_cast<const char*>(K) + (tok0 * H + h) * (int64_t)d_k * (KD == OP_F32 ? 4 : 2);
    TRIINV_PER_WAVE(w, (team64_solve<KD, OP, METHOD, DKS, NRHS, W>(key_lds, area, Kc, (int64_t)H * d_k, beta + tok0 * H + h, g ? g + tok0 * H + h : nullptr, rhs,
                                                                   tok0, h, H, pos.valid, aux, ln)))
}

// Per-channel gate.
template <int OP, int METHOD, int NRHS, int W>
__device__ __forceinline__ void team64_solve_channels(const Team& team, const float* bc, const RhsList& rhs, int64_t tok0, int h, int H, int valid, int aux, Lane ln)
{
    Team64Apply<OP, W, NRHS> apply(rhs, tok0, h, H, valid, ln);
    apply.issue(0);
    team64_from_channels<OP, METHOD, W>(team, bc, H, valid, aux, ln, [&](float* strip) { apply(strip); });
}

template <int OP, int METHOD, int NRHS>
__global__ __launch_bounds__(256) void k_kda_tri_solve_team64(const void* __restrict__ K, const float* __restrict__ beta, const float* __restrict__ g, RhsList rhs,
                                                              int64_t n_chunk, SolveMap<NRHS == 1> map, int H, int d_k, int k_dt, int aux)
{
    arguments_together(n_chunk, K, beta, g, rhs.r[0].X, map);
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
    TRIINV_PER_WAVE(team.w, (team64_solve_channels<OP, METHOD, NRHS, W>(team, beta + tok0 * H + h, rhs, tok0, h, H, pos.valid, aux, ln)))
}

// Scalar / no-gate kinds, any d_k.
template <int KD, int OP, int METHOD, int NRHS, int W>
__device__ __forceinline__ void team64_solve_products(const Team& team, const float* bc, const float* gc, const RhsList& rhs, int64_t tok0, int h, int H, int valid,
                                                      int aux, Lane ln)
{
    Team64Apply<OP, W, NRHS> apply(rhs, tok0, h, H, valid, ln);
    apply.issue(0);
    team64_from_products<KD, OP, METHOD, W>(team, bc, gc, H, valid, aux, ln, [&](float* strip) { apply(strip); });
}

template <int KD, int OP, int METHOD, int NRHS>
__global__ __launch_bounds__(256) void k_gdn_any_dk_tri_solve_team64(const void* __restrict__ K, const float* __restrict__ beta, const float* __restrict__ g,
                                                              RhsList rhs, int64_t n_chunk, SolveMap<NRHS == 1> map, int H, int d_k, int aux)
{
    arguments_together(n_chunk, K, beta, g, rhs.r[0].X, map);
    __shared__ __attribute__((aligned(16))) char lds[Team64Loop<KD, OP, METHOD, false>::BYTES];
    const uint32_t m = blockIdx.x, bc = m / (uint32_t)H;
    const int h = (int)(m - bc * (uint32_t)H);
    const ChunkPos pos = locate_chunk<64>(map, bc);
    const int64_t tok0 = pos.tok0, row_stride = (int64_t)H * d_k;
    const Lane ln = lane_id();
    const void* const Kc = static_cast<const char*>(K) + (tok0 * H + h) * (int64_t)d_k * (KD == OP_F32 ? 4 : 2);
    const Team team = this_team(lds);
    team_gram_products<KD, 4, METHOD, KD != OP_F32, false>(Kc, KD == OP_F16, nullptr, row_stride, d_k / 32, ln, pos.valid, team);
    TRIINV_PER_WAVE(team.w, (team64_solve_products<KD, OP, METHOD, NRHS, W>(team, beta + tok0 * H + h, g ? g + tok0 * H + h : nullptr, rhs, tok0, h, H, pos.valid,
                                                                            aux, ln)))
}

}  // namespace triinv
