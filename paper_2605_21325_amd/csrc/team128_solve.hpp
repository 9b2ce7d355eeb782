// The teams of team128.hpp with the inverse applied instead of stored (W_k = T diag(s_k) X_k, blocked and mixed recursion): wave w forms tile row w of W,
// from its strip of T and tile rows 0 .. w of X, which it requested ahead of the recursion.
#pragma once
#include "solve.hpp"
#include "team128.hpp"

namespace triinv {

// Four elements of T times their columns' scales as an operand.  With f16 the two-wavefront kernels scale the inverse's left half element by element
// (TileLds::narrow), which the compiler makes one operation with one rounding of each product, and the rest of it in pairs, which is rounded to fp32 first:
// the same here, for the same bits.
template <int OP, bool LEFT> __device__ __forceinline__ Opnd<OP> scaled_operand(v4f t, v4f s)
{
    if constexpr (OP != OP_F16 || !LEFT) {
        return pack<OP>(t * s);
    } else {
        uint32_t u[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            _Float16 x = (_Float16)(t[r] * s[r]);
            asm("" : "+v"(x));  // (not in pairs)
            u[r] = __builtin_bit_cast(uint16_t, x);
        }
        return {__builtin_bit_cast(v4h, v2u{u[0] | u[1] << 16, u[2] | u[3] << 16})};
    }
}

// The right-hand sides, as wave w of a team takes them: the first requested early, the others one after the other.
template <class LY, int OP, int NRHS> struct Team128Apply {
    static constexpr int VEC = RhsX<OP, 8, true>::VEC;
    const RhsList& rhs;
    int64_t tok0;
    int h, H, valid, w;
    Lane ln;
    float* scales;       // 128 floats of LDS
    RhsX<OP, 8, true> x;
    float scale[2];      // of tokens lane, lane + 64; x.s_q is not used (32 registers)

    __device__ __forceinline__ Team128Apply(char* lds, const RhsList& rhs_, int64_t tok0_, int h_, int H_, int valid_, int w_, Lane ln_)
        : rhs(rhs_), tok0(tok0_), h(h_), H(H_), valid(valid_), w(w_), ln(ln_), scales(reinterpret_cast<float*>(lds + LY::SMALL) + w_ * LY::SMALL_FLOATS)
    {
    }
    __device__ __forceinline__ void issue(int gi)  // tile rows 0 .. w
    {
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (j <= w) x.issue(gi, j, j + 1);
    }
    __device__ __forceinline__ void start(int k)
    {
        Lane l = ln;
        asm volatile("" : "+v"(l.q), "+v"(l.n));  // (what the sides' addresses have in common is not worth registers from one to the other)
        x.init(rhs.r[k], tok0, h, H, valid, l);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int at = 16 * l.q + l.n + 64 * t, row = at < valid ? at : valid - 1;
            scale[t] = rhs.r[k].scale ? rhs.r[k].scale[(tok0 + row) * H + h] : 1.f;
        }
        issue(0);
    }
    __device__ __forceinline__ void operator()(const float* strip)
    {
        const int lane = 16 * ln.q + ln.n;
#pragma unroll
        for (int k = 0; k < NRHS; ++k) {
            if (k > 0) {
                __builtin_amdgcn_sched_barrier(0);
                start(k);
            }
            scales[lane] = scale[0];
            scales[lane + 64] = scale[1];
            wave_lds_sync();
            Opnd<OP> Top[8];  // T orientation: columns scaled by s in fp32, then rounded to the operand type
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (j <= w) {
                    const v4f t = *reinterpret_cast<const v4f*>(&strip[ln.n * LY::STRIP_LD + 16 * j + 4 * ln.q]);
                    const v4f s = *reinterpret_cast<const v4f*>(&scales[16 * j + 4 * ln.q]);
                    Top[j] = j < 4 ? scaled_operand<OP, true>(t, s) : scaled_operand<OP, false>(t, s);
                }
            wave_lds_sync();
            __builtin_amdgcn_sched_barrier(0);
            const int n_group = x.n_group();
#pragma unroll 1
            for (int gi = 0;;) {
                v4f acc[VEC];
#pragma unroll
                for (int c = 0; c < VEC; ++c) acc[c] = zero4();
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (j <= w) {
#pragma unroll
                        for (int c = 0; c < VEC; ++c) acc[c] = tn<OP>(Top[j], x_operand<OP>(x.raw[j], c), acc[c]);
                        __builtin_amdgcn_sched_barrier(0);  // (one tile row's operands at a time)
                    }
                const int done = gi++;
                if (gi < n_group) issue(gi);
                x.store(done, w, acc);
                if (gi >= n_group) break;
            }
        }
    }
};

// MERGE_T: see team128_recursion.
template <int KD, int OP, int METHOD, int DKS, int NRHS, bool MERGE_T>
__global__ __launch_bounds__(512) void k_gdn_tri_solve_team128(const void* __restrict__ K, const float* __restrict__ beta, const float* __restrict__ g, RhsList rhs,
                                                               int64_t n_chunk, SolveMap<NRHS == 1> map, int H, int d_k, int aux)
{
    arguments_together(n_chunk, K, beta, g, rhs.r[0].X, map);
    typedef Team128Lds<KD, OP, METHOD, DKS> LY;
    __shared__ __attribute__((aligned(16))) char lds[LY::BYTES];
    const uint32_t m = blockIdx.x, bc = m / (uint32_t)H;
    const int h = (int)(m - bc * (uint32_t)H);
    const ChunkPos pos = locate_chunk<128>(map, bc);
    const int64_t tok0 = pos.tok0;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const Lane ln = lane_id();
    const void* const Kc = static_cast<const char*>(K) + (tok0 * H + h) * (int64_t)d_k * (KD == OP_F32 ? 4 : 2);
    Team128Apply<LY, OP, NRHS> apply(lds, rhs, tok0, h, H, pos.valid, w, ln);
    const auto own = team128_tiles<KD, OP, METHOD, DKS, MERGE_T>(lds, Kc, (int64_t)H * d_k, beta + tok0 * H + h, g ? g + tok0 * H + h : nullptr, H, pos.valid, w,
                                                                 ln, [&]() { apply.start(0); });
    team128_recursion<LY, OP, METHOD, MERGE_T>(lds, own, aux, w, ln, [&](const float* strip) { apply(strip); });
}

// Per-channel gate: X is requested once keys and gates have left their registers.
template <int OP, int METHOD, bool K16, int NRHS>
__global__ __launch_bounds__(512) void k_kda_tri_solve_team128(const void* __restrict__ K, const float* __restrict__ beta, const float* __restrict__ g, RhsList rhs,
                                                               int64_t n_chunk, SolveMap<NRHS == 1> map, int H, int d_k, int k_dt, int aux)
{
    arguments_together(n_chunk, K, beta, g, rhs.r[0].X, map);
    typedef Team128KdaLds<OP, METHOD> LY;
    __shared__ __attribute__((aligned(16))) char lds[LY::BYTES];
    const uint32_t m = blockIdx.x, bc = m / (uint32_t)H;
    const int h = (int)(m - bc * (uint32_t)H);
    const ChunkPos pos = locate_chunk<128>(map, bc);
    const int64_t tok0 = pos.tok0, e0 = (tok0 * H + h) * (int64_t)d_k;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const Lane ln = lane_id();
    const auto own = team128_kda_tiles<OP, METHOD, K16>(lds, static_cast<const char*>(K) + e0 * (K16 ? 2 : 4), k_dt == OP_F16, g + e0, (int64_t)H * d_k, d_k,
                                                        beta + tok0 * H + h, H, pos.valid, w, ln);
    Team128Apply<LY, OP, NRHS> apply(lds, rhs, tok0, h, H, pos.valid, w, ln);
    apply.start(0);
    team128_recursion<LY, OP, METHOD, false>(lds, own, aux, w, ln, [&](const float* strip) { apply(strip); });
}

}  // namespace triinv
