// Host-side launch table: one launcher per (C, operand type) pair, each compiled in its own
// translation unit (inst.hip with TRIINV_INST_NB / TRIINV_INST_OP set) so the build parallelises.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <tuple>
#include <type_traits>
#include <utility>
#include "../../include/triinv.h"
#include "chunk_map.hpp"

namespace triinv {

struct TriInvArgs {
    const void* A;
    float* T;
    int64_t n_mat;
    int in_dt;
    int method;
    hipStream_t stream;
    bool refine;  // one iterative-refinement step after the method
    int iters;    // Newton-Schulz iteration count; for the mixed recursion: refinement steps on the 16 x 16 blocks
    int out_dt;   // element type of T: 0 fp32, 1 fp16, 2 bf16
    bool shuffle; // forward substitution: broadcast A by wavefront shuffles (C = 64)
    bool dry = false;  // only report whether the combination is built; launch nothing
};

struct GdnArgs {
    const void* K;
    const float* beta;
    const float* g;  // null for the no-gate kind
    float* T;
    int64_t n_mat;
    int64_t n_chunk;  // total number of chunks
    ChunkMap map;     // where each chunk's tokens are
    int H;
    int d_k;
    int k_dt;
    int gate;
    int method;
    hipStream_t stream;
    bool refine;
    int iters;
    int out_dt;
    bool dry = false;  // only report whether the combination is built; launch nothing
};

// gdn_chunk_tri_solve: the fused arguments (T unused) plus the right-hand sides.
struct SolveArgs {
    GdnArgs f;
    int n_rhs;             // 1 or 2 right-hand sides sharing the inverse
    const void* X[2];      // [tokens][H][d_x], element type = operand type
    const float* scale[2]; // [tokens][H] or null
    void* W[2];            // [tokens][H][d_x]
    int d_x[2];
};

// The chunk stride of the few-heads workgroup map of the fused kernels (0 = the many-heads map): see fused_matrix_index.
inline int head_spread(int H) { return H >= 8 ? 0 : (H >= 4 ? 1 : 4 / H); }

// Grid of the fused kernels that put `waves` wavefronts, a matrix each, into a workgroup.  Up to two matrices per compute unit (256 of
// them) a workgroup holds one: four wavefronts would load their keys and store their results through one compute unit while
// others have nothing to do.  Kernel time at C = 64, four / one to a workgroup: 256 matrices 6.4 / 5.4 us (bf16), 16.1 / 11.6
// (per-channel gate), 13.9 / 11.7 (fp32 keys and operands), applied to two right-hand sides 11.2 / 9.3; 512 6.5 / 6.0 and 17.1 / 13.3; 1024
// 7.6 / 7.5 and 18.2 / 18.8; 1536 9.3 / 12.2.  (Recursions at C = 64 with few matrices go to the teams below first.)
constexpr int ONE_WAVE_PER_GROUP = -1;  // in place of the spread
constexpr int64_t FEW_MATRICES = 512;
// The channel loops (per-channel gate, head dimensions without a kernel of their own) share a matrix of such a call between four
// wavefronts where there is more than one k-step (32 channels).
constexpr int TEAM_WAVES = 4;
inline bool by_team(int64_t n_mat, int d_k) { return n_mat <= FEW_MATRICES && d_k > 32; }
// C = 128, head dimensions without a kernel of their own (fp32 keys of 128 channels with fp32 operands and forward substitution among them): up to one team per
// compute unit.  256 matrices, one wavefront / a team: fp32 keys, d_k = 128, forward substitution 40.9 / 28.2 us (8 of them 40.9 / 27.3), blocked recursion
// with fp32 operands 44.3 / 27.5, d_k = 256, 16-bit operands, mixed 61.9 / 28.6 (172, blocked: 54.4 / 21.1); bf16 keys, d_k = 256 16.6 / 13.3, d_k = 96 17.7 /
// 17.5.  512, two teams a compute unit: 45.3 / 35.5, 48.4 / 54.0, 60.6 / 44.4 (blocked), 20.9 / 25.9.
inline bool by_team128(int64_t n_mat, int d_k) { return n_mat <= FEW_MATRICES / 2 && d_k > 32; }
// fp32 keys of 128 channels go the same way at C = 64 (methods without a team64 kernel) although that head dimension has a kernel of its own: their Gram products are fp32
// matrix instructions, 6 of the 11.7 us of such a call, and each diagonal tile's products are formed once there.  Up to one team per compute unit:
// 256 matrices 11.8 / 9.6 us (own kernel / team; bf16 operands 9.7 / 8.0, one right-hand side applied 17.3 / 15.8), 512 12.8 / 12.3 and
// 10.7 / 10.3.  (64 channels, half the products, keep their kernel: 256 matrices 9.2 / 8.6 and 7.4 / 6.8, 512 10.1 / 10.1 and 8.1 / 8.3.)
constexpr int FP32_KEYS_TEAM_DK = 128;
inline bool fp32_keys_by_team(int64_t n_mat, int d_k, int C) { return C == 64 && d_k == FP32_KEYS_TEAM_DK && n_mat <= FEW_MATRICES / 2; }
// C = 64, d_k = 64 or 128, blocked, mixed and direct-leaf recursion: four wavefronts to a matrix from the keys to the store (team64.hpp), up to three
// teams per compute unit (fp32 keys of 128 channels: two fit, and more than 512 matrices take two rounds; still level or ahead: one wavefront / a team, 520
// matrices 14.2 / 13.5 us, with 16-bit operands 12.4 / 12.3, 640 14.1 / 13.8 and 12.4 / 12.4, 768 14.2 / 13.7 and 12.5 / 12.5, of one head 640 14.3 / 13.0 and
// 12.4 / 11.8); the direct leaves, whose one chain of vector instructions nothing shortens, up to one.  One wavefront to a matrix / a team: 8
// matrices bf16 4.9 / 4.0 us, fp32 keys and operands 8.9 / 5.2; 256: 5.1 / 4.4, fp32 operands 7.4 / 5.2, fp32 keys and operands of 128 channels (whose
// tiles a team formed before too) 9.5 / 6.7, direct leaves 5.0 / 4.9; 512: 5.6 / 5.3, 8.0 / 6.6, 12.4 / 9.3, 5.8 / 5.9; 768: 6.8 / 6.3, 9.2 / 8.1; 1024:
// 7.6 / 8.3, 10.0 / 10.2, 15.6 / 17.3.
inline bool by_team64(int64_t n_mat, bool direct) { return n_mat <= (direct ? 256 : 768); }
// Applied to right-hand sides (team64_solve.hpp).  One / two of 128 columns, 256 matrices: bf16 6.7 / 5.3 and 8.9 / 6.5, fp32 operands 12.7 / 7.5 and 18.9 /
// 10.7; 512: 7.6 / 7.1, 9.9 / 9.1, 14.4 / 11.5; 768: 9.1 / 8.9, 11.5 / 16.0, 17.0 / 16.0, 25.4 / 28.2.
inline bool solve_by_team64(int64_t n_mat) { return n_mat <= FEW_MATRICES; }
// C = 128, the same, eight wavefronts to a matrix (team128.hpp), whose 112 to 150 KB of LDS let a compute unit hold one team.  Kernel of the larger calls /
// a team: 8 matrices bf16 7.5 / 7.1 us, fp32 operands 17.6 / 9.1; 256: 9.0 / 9.0, fp16 mixed 9.3 / 8.8, fp32 operands 19.0 / 11.1, mixed 19.7 / 11.3, direct
// leaves 17.0 / 11.1, fp32 keys of 64 channels 25.8 / 13.1, of 128 with 16-bit operands 21.7 / 14.4.
inline bool recursion_by_team128(int64_t n_mat) { return n_mat <= 256; }
// Applied to right-hand sides (team128_solve.hpp), kernel of the larger calls / a team.  8 matrices, one side of 128 columns: bf16 11.3 / 9.8 us, fp32
// operands 36.3 / 16.3; 256: bf16 12.2 / 10.6 (two sides 17.0 / 13.9), fp16 of 64 channels 11.3 / 10.5, fp32 operands 37.1 / 17.8 (42.6 / 27.6), fp32 keys
// with 16-bit operands 24.4 / 16.2.
inline bool solve_by_team128(int64_t n_mat) { return n_mat <= 256; }
// The per-channel gate at C = 128 (two wavefronts / a team, d_k = 128).  8 matrices bf16 14.5 / 12.1 us, fp32 keys and operands 32.4 / 19.5; 256: bf16 16.4 /
// 14.5, applied 20.0 / 15.5 (two sides 27.2 / 19.6), fp32 operands 34.8 / 21.8, applied 49.5 / 28.2, fp16 mixed of 64 channels 11.7 / 10.7; 128 of 256 channels
// 23.4 / 17.6, of 32 8.3 / 7.7.
inline bool channels_by_team128(int64_t n_mat) { return n_mat <= 256; }
// Newton-Schulz at C = 128: eight wavefronts in place of four, as long as a compute unit has one matrix.  Four / eight, 16 matrices with fp32 operands 71 /
// 50 us, 64 with bf16 24.0 / 18.3; 256: fp32 72 / 53, bf16 25.7 / 20.7, standalone 24.1 / 18.7, fp32 70 / 51.  Per-channel gate (the two of a pair of tile
// rows form the same tiles), 64 bf16 of 256 channels 33.3 / 31.7; kernel of larger calls before X was turned by LDS reads / eight: 16 fp32 80 / 63, 256 bf16
// 31.1 / 26.4, of 64 channels 28.6 / 22.6.  (One tile row a wave gave nothing, 69 of 70 us: the wave of the last row has as much to do as one of four.)
inline bool newton_by_eight(int64_t n_mat) { return n_mat <= 256; }
struct FusedGrid {
    unsigned groups, threads;
    int spread;
    bool few() const { return spread < 0; }
};
inline FusedGrid fused_grid(int64_t n_mat, int H, int waves)
{
    if (waves > 1 && n_mat <= FEW_MATRICES) return {(unsigned)n_mat, 64u, ONE_WAVE_PER_GROUP};
    return {(unsigned)((n_mat + waves - 1) / waves), 64u * waves, waves > 1 ? head_spread(H) : 0};
}

// Lengths of packed sequences go with the arguments of the storing kernels but for the Neumann product, b0 = 32 and the refinement step, some of which lose
// a wavefront per SIMD by the registers of the search (refined Neumann product, C = 64, d_k = 64, 4096 matrices: 20.9 -> 23.3 us).
constexpr bool lengths_in_arguments(int method, bool refine) { return !refine && method != TRIINV_NEUMANN && method != TRIINV_MIXED_B32; }
// Single kernels that are slower by it than a packed call gains, with all calls that are not packed.
// Per-channel gate, forward substitution at C = 128 (all of the register file; offsets / lengths, and the arguments loaded at once): 1024 matrices of bf16 keys,
// d_k = 128, 61.9 / 66.1 us, 4096 241 / 259 (fp32 keys 277 / 294).
constexpr bool kda_lengths(int C, int method, bool refine) { return lengths_in_arguments(method, refine) && !(method == TRIINV_FWD_SUBST && C == 128); }
// Channels of a kernel with this many k-steps.  (A function: written out with the operand codes, whose enumeration has no name, the type of a kernel's
// parameter has another name on the host than on the device, and the launch aborts.)
constexpr int key_channels(int k_dtype, int k_steps) { return k_steps * (k_dtype == TRIINV_F32 ? 16 : 32); }
// Forward substitution of fp32 keys of 64 channels at C = 64 (offsets / lengths): 3000 matrices 21.9 / 23.7 us, 8192 53.5 / 54.5.  Newton-Schulz at C <= 64,
// 16-bit keys and operands: 600 matrices of C = 32 4.9 / 5.3 us, 3000 7.5 / 7.7, 600 of C = 16 3.8 / 4.0, of C = 64 10.8 / 11.3, 3000 20.9 / 21.9.  The
// mixed recursion at C <= 64, every type: 64 matrices of C = 32, bf16, 3.7 / 4.1 us, fp32 keys and operands 5.1 / 5.5, 3000 7.4 / 7.6 and 11.2 / 11.4, 900 of C =
// 16 3.6 / 3.75, 800 of C = 64 6.8 / 7.0 and 11.0 / 11.5 (up to 768 it is a team's; blocked recursion, direct leaves and forward substitution otherwise level).
constexpr bool gdn_lengths(int C, int k_dtype, int d_k, int method, bool refine)
{
    return lengths_in_arguments(method, refine) && !(method == TRIINV_FWD_SUBST && C == 64 && k_dtype == TRIINV_F32 && d_k == 64) &&
           !(method == TRIINV_NEWTON_SCHULZ && C <= 64) && !(method == TRIINV_MIXED && C <= 64);
}
// The inverse applied to one right-hand side.  fp16 keys of 64 channels at C = 64, blocked recursion (offsets / lengths): 3000 matrices 19.9 / 21.7 us, 3500
// 23.1 / 24.3, 8192 49.6 / 50.4; bf16 keys 21.7 / 21.9, 128 channels 22.5 / 22.8, mixed recursion 21.1 / 21.1.  C = 128 with 16-bit operands: this kernel stands in
// for rows too long for the one on two wavefronts and fills the register file.
constexpr bool solve_lengths(int C, int k_dtype, int d_k, int op, int method)
{
    return C == 128 ? op == TRIINV_F32 : !(C == 64 && k_dtype == TRIINV_F16 && d_k == 64 && op == TRIINV_F16 && method == TRIINV_BLOCK_RECURSIVE);
}

// Launcher return codes.
enum : int { LAUNCHED = 0, NOT_BUILT = 1, LAUNCH_FAILED = 2 };

// Whether a kernel's parameter holds all of this argument.
template <class Param, class Arg> inline bool holds(const Arg& a)
{
    if constexpr (std::is_same_v<Arg, ChunkMap>)
        return Param::takes(a);
    else
        return (void)a, true;
}

// One kernel launch whose own status is returned (the runtime's sticky per-thread error state, which may hold an
// unrelated earlier error of the caller, is neither read nor cleared).  The arguments are converted to the kernel's
// exact parameter types first.  dry: report LAUNCHED without launching.  Lengths of packed sequences for a kernel that cannot be given them: NOT_BUILT.
template <class... KArgs, class... Args, size_t... I>
inline int launch_kernel_impl(void (*kernel)(KArgs...), dim3 grid, dim3 block, unsigned lds_bytes, hipStream_t stream,
                              std::index_sequence<I...>, Args&&... args)
{
    std::tuple<KArgs...> vals{static_cast<KArgs>(std::forward<Args>(args))...};
    void* ptrs[sizeof...(KArgs)] = {(void*)&std::get<I>(vals)...};
    return hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, ptrs, lds_bytes, stream) == hipSuccess ? LAUNCHED : LAUNCH_FAILED;
}
template <class... KArgs, class... Args>
inline int launch_kernel(bool dry, void (*kernel)(KArgs...), dim3 grid, dim3 block, unsigned lds_bytes, hipStream_t stream, Args&&... args)
{
    static_assert(sizeof...(KArgs) == sizeof...(Args), "one argument per kernel parameter");
    if (!(holds<KArgs>(args) && ...)) return NOT_BUILT;
    if (dry) return LAUNCHED;
    return launch_kernel_impl(kernel, grid, block, lds_bytes, stream, std::index_sequence_for<KArgs...>{}, std::forward<Args>(args)...);
}

// Every launcher returns one of the codes above.
#define TRIINV_DECL(NB, OP)                                  \
    int launch_tri_inv_nb##NB##_op##OP(const TriInvArgs& a); \
    int launch_gdn_nb##NB##_op##OP(const GdnArgs& a);        \
    int launch_gdn_nb##NB##_op##OP##_fwd(const GdnArgs& a);
TRIINV_DECL(1, 0)
TRIINV_DECL(1, 1)
TRIINV_DECL(1, 2)
TRIINV_DECL(2, 0)
TRIINV_DECL(2, 1)
TRIINV_DECL(2, 2)
TRIINV_DECL(4, 0)
TRIINV_DECL(4, 1)
TRIINV_DECL(4, 2)
TRIINV_DECL(8, 0)
TRIINV_DECL(8, 1)
TRIINV_DECL(8, 2)
#undef TRIINV_DECL
#define TRIINV_DECL_SOLVE(NB) \
    int launch_solve_nb##NB##_op0(const SolveArgs& a); \
    int launch_solve_nb##NB##_op1(const SolveArgs& a); \
    int launch_solve_nb##NB##_op2(const SolveArgs& a);
TRIINV_DECL_SOLVE(1)
TRIINV_DECL_SOLVE(2)
TRIINV_DECL_SOLVE(4)
TRIINV_DECL_SOLVE(8)
#undef TRIINV_DECL_SOLVE
int launch_tri_inv_nb1_op0_fwd(const TriInvArgs& a);
int launch_tri_inv_nb2_op0_fwd(const TriInvArgs& a);
int launch_tri_inv_nb4_op0_fwd(const TriInvArgs& a);
int launch_tri_inv_nb8_op0_fwd(const TriInvArgs& a);

}  // namespace triinv
