// 16 x 16 register tiles and the one matrix-core primitive everything is built from (gfx950).
//
// A logical 16 x 16 fp32 matrix M lives in 4 VGPRs of one 64-lane wavefront in the accumulator
// layout of the 16x16 MFMA instructions: lane l = 16*q + n (q = l / 16, n = l % 16) holds
//     v[r] = M[4*q + r][n],  r = 0..3.
// The same four registers, narrowed to the operand type, are a valid B operand of M (contraction
// over M's ROW index) and a valid A operand of M^T.  Hence the single primitive
//     tn(X, Y) = X^T * Y          (X, Y, result all in the layout above)
// needs no cross-lane movement between dependent products.  A matrix that must act as a LEFT
// factor is therefore kept transposed ("T orientation": the tile registers hold M^T), a RIGHT
// factor as is ("N orientation").
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace triinv {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef short v4s __attribute__((ext_vector_type(4)));
typedef _Float16 v4h __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef short v8s __attribute__((ext_vector_type(8)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

enum : int { OP_F32 = 0, OP_F16 = 1, OP_BF16 = 2 };

struct Lane {
    int q;  // lane / 16 : row group (rows 4q..4q+3 of a tile)
    int n;  // lane % 16 : column of a tile
};

__device__ __forceinline__ Lane lane_id()
{
    int l = __lane_id();
    return Lane{l >> 4, l & 15};
}

// Two fp32 -> two bf16 / fp16 in one register, round to nearest even (one v_cvt_pk_bf16_f32 on gfx950).
__device__ __forceinline__ uint32_t pack2_bf16(float a, float b)
{
    const v2f f = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, v2bf));
}
__device__ __forceinline__ uint32_t pack2_f16(float a, float b)
{
    const v2f f = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, v2h));
}

__device__ __forceinline__ float bf16_to_f32(uint16_t b)
{
    return __builtin_bit_cast(float, ((uint32_t)b) << 16);
}

__device__ __forceinline__ float f16_to_f32(uint16_t h)
{
    return (float)__builtin_bit_cast(_Float16, h);
}

// Packed matrix-core operand of one tile.
template <int OP> struct Opnd;
template <> struct Opnd<OP_F32> { v4f x; };
template <> struct Opnd<OP_F16> { v4h x; };
template <> struct Opnd<OP_BF16> { v4s x; };

template <int OP> __device__ __forceinline__ Opnd<OP> pack(v4f t);
template <> __device__ __forceinline__ Opnd<OP_F32> pack<OP_F32>(v4f t) { return {t}; }
template <> __device__ __forceinline__ Opnd<OP_F16> pack<OP_F16>(v4f t)
{
    const v2u u = {pack2_f16(t[0], t[1]), pack2_f16(t[2], t[3])};
    return {__builtin_bit_cast(v4h, u)};
}
template <> __device__ __forceinline__ Opnd<OP_BF16> pack<OP_BF16>(v4f t)
{
    const v2u u = {pack2_bf16(t[0], t[1]), pack2_bf16(t[2], t[3])};
    return {__builtin_bit_cast(v4s, u)};
}

// Element masks of one tile as bit patterns on the packed operand: keeping an element is an AND
// with all ones, dropping it an AND with zero (which also kills NaN / Inf).
template <int OP> struct Mask;
template <> struct Mask<OP_F32> { v4u m; };
template <> struct Mask<OP_F16> { v2u m; };
template <> struct Mask<OP_BF16> { v2u m; };

template <int OP> __device__ __forceinline__ Mask<OP> make_mask(bool k0, bool k1, bool k2, bool k3)
{
    Mask<OP> o;
    if constexpr (OP == OP_F32) {
        o.m = v4u{k0 ? ~0u : 0u, k1 ? ~0u : 0u, k2 ? ~0u : 0u, k3 ? ~0u : 0u};
    } else {
        o.m = v2u{(k0 ? 0xffffu : 0u) | (k1 ? 0xffff0000u : 0u), (k2 ? 0xffffu : 0u) | (k3 ? 0xffff0000u : 0u)};
    }
    return o;
}

template <int OP> __device__ __forceinline__ Opnd<OP> masked(Opnd<OP> x, Mask<OP> k)
{
    if constexpr (OP == OP_F32) {
        return {__builtin_bit_cast(v4f, __builtin_bit_cast(v4u, x.x) & k.m)};
    } else {
        Opnd<OP> o;
        o.x = __builtin_bit_cast(decltype(o.x), __builtin_bit_cast(v2u, x.x) & k.m);
        return o;
    }
}

// -x: a sign flip on the packed operand (two instructions for the 16-bit types, half of what negating the fp32 tile costs).
template <int OP> __device__ __forceinline__ Opnd<OP> negated(Opnd<OP> x)
{
    if constexpr (OP == OP_F32) {
        return {-x.x};
    } else {
        Opnd<OP> o;
        o.x = __builtin_bit_cast(decltype(o.x), __builtin_bit_cast(v2u, x.x) ^ v2u{0x80008000u, 0x80008000u});
        return o;
    }
}

// acc + X^T * Y   (x packed from X, y packed from Y)
template <int OP> __device__ __forceinline__ v4f tn(Opnd<OP> x, Opnd<OP> y, v4f acc);
template <> __device__ __forceinline__ v4f tn<OP_F32>(Opnd<OP_F32> x, Opnd<OP_F32> y, v4f acc)
{
    // 16x16x4 fp32: k slot q of step r stands for contraction index 4q + r on both operands
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x.x[0], y.x[0], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x.x[1], y.x[1], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x.x[2], y.x[2], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x.x[3], y.x[3], acc, 0, 0, 0);
    return acc;
}
template <> __device__ __forceinline__ v4f tn<OP_F16>(Opnd<OP_F16> x, Opnd<OP_F16> y, v4f acc)
{
    return __builtin_amdgcn_mfma_f32_16x16x16f16(x.x, y.x, acc, 0, 0, 0);
}
template <> __device__ __forceinline__ v4f tn<OP_BF16>(Opnd<OP_BF16> x, Opnd<OP_BF16> y, v4f acc)
{
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(x.x, y.x, acc, 0, 0, 0);
}

// acc + sum over k in [lo, hi] of X(k)^T * Y(k); live(k): a wave-uniform run-time test that may drop terms whose tiles
// are known to hold zeros.
template <int OP, class FX, class FY, class Live>
__device__ __forceinline__ v4f tn_sum_if(int lo, int hi, FX x, FY y, Live live, v4f acc)
{
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        if (k < lo || k > hi) continue;
        if (live(k)) acc = tn<OP>(x(k), y(k), acc);
    }
    return acc;
}
template <int OP, class FX, class FY> __device__ __forceinline__ v4f tn_sum(int lo, int hi, FX x, FY y, v4f acc)
{
    return tn_sum_if<OP>(lo, hi, x, y, [](int) { return true; }, acc);
}

__device__ __forceinline__ v4f zero4() { return v4f{0.f, 0.f, 0.f, 0.f}; }

// The 16 x 16 identity in tile layout (either orientation).
__device__ __forceinline__ v4f identity_tile(Lane ln)
{
    v4f v;
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = 4 * ln.q + r == ln.n ? 1.f : 0.f;
    return v;
}

// Two packed 16-bit tiles as one operand of the 32-deep instructions (gfx950): contraction slot 8 q + e stands for row
// 4 q + e of the first tile (e < 4) or row 4 q + e - 4 of the second, the same on both operands, so the halves are just
// the two packed tiles.  A chain of these instructions holds no 16-deep ones: the two kinds feeding one accumulator were
// seen to give wrong tiles.
template <int OP> struct PairOp {
    v4u u;
    __device__ __forceinline__ void set(int half, Opnd<OP> x)
    {
        const v2u w = __builtin_bit_cast(v2u, x.x);
        u[2 * half] = w[0];
        u[2 * half + 1] = w[1];
    }
    __device__ __forceinline__ Opnd<OP> get(int half) const
    {
        Opnd<OP> o;
        o.x = __builtin_bit_cast(decltype(o.x), v2u{u[2 * half], u[2 * half + 1]});
        return o;
    }
};
template <int OP> __device__ __forceinline__ v4f tn_pair(PairOp<OP> x, PairOp<OP> y, v4f acc)
{
    if constexpr (OP == OP_F16)
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h, x.u), __builtin_bit_cast(v8h, y.u), acc, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, x.u), __builtin_bit_cast(v8bf, y.u), acc, 0, 0, 0);
}

// The terms k = 2 p, 2 p + 1 of a tile (i, j) of a product of lower triangular matrices, sum over j <= k <= i.  Where both are
// terms: one 32-deep instruction into acc.  Where one is: a 16-deep one, into `odd` if the tile has pairs too (mixed_terms;
// started from zero here, to be added to acc at the end), into acc otherwise.  A 32-deep instruction with a zero in place of the
// other tile would take as long, but that tile's partner is a real one, from outside the sum: where it is not finite, its
// product with zero is NaN.
__host__ __device__ constexpr bool has_pairs(int i, int j) { return (i + 1) / 2 > (j + 1) / 2; }
__host__ __device__ constexpr bool mixed_terms(int i, int j) { return has_pairs(i, j) && (j % 2 == 1 || i % 2 == 0); }
template <int OP> __device__ __forceinline__ void pair_term(int p, int i, int j, const PairOp<OP>& x, const PairOp<OP>& y, v4f& acc, v4f& odd)
{
    const bool low = j <= 2 * p && 2 * p <= i, high = j <= 2 * p + 1 && 2 * p + 1 <= i;
    if (low && high)
        acc = tn_pair<OP>(x, y, acc);
    else if (low || high) {
        const bool first = p == j / 2 && j % 2 == 1;  // (the other single term, if there is one, is the last)
        if (mixed_terms(i, j))
            odd = tn<OP>(x.get(high), y.get(high), first || j % 2 == 0 ? zero4() : odd);
        else
            acc = tn<OP>(x.get(high), y.get(high), acc);
    }
}

// An fp32 tile as the sum of three bf16 tiles, x = h + m + l: h = bf16(x), m = bf16(x - h), l = x - h - m, which is exact
// (24 = 3 x 8 bits; both differences are exact, and what remains after m has at most 8 bits) for |x| between 2^-110, below
// which l runs into bf16's smallest subnormal, and 3.39e38, the largest bf16, above which h is infinite and the sum NaN
// (split3_any takes every finite x).  The product of two such tiles is hh + hm + mh + hl + lh + mm, accumulated in fp32; what is
// left out, ml + lm + ll, is at most 2^-24 |x| |y| (|m| <= 2^-8 |x|, |l| <= 2^-17 |x|; both at once is rare: root mean square 2^-27.5
// over random mantissas), where an fp32 multiply-add rounds its sum, not the product.  Whole iterations are no less accurate for it (see
// newton_schulz): three 32-deep bf16 instructions of 16 cycles against four 16x16x4 fp32 instructions of 32.
// Splitting costs 22 vector instructions a tile, so it pays where an operand is used several times.
// The parts sit side by side in the order m h l, so that two overlapping windows of either operand feed the instructions:
//   (m h) . (m h) = mm + hh,   (m h) . (h l) = mh + hl,   (h l) . (m h) = hm + lh.
typedef uint32_t v6u __attribute__((ext_vector_type(6)));
struct Split3 {
    v6u u;
    __device__ __forceinline__ Opnd<OP_BF16> m() const { return {__builtin_bit_cast(v4s, v2u{u[0], u[1]})}; }
    __device__ __forceinline__ Opnd<OP_BF16> h() const { return {__builtin_bit_cast(v4s, v2u{u[2], u[3]})}; }
    __device__ __forceinline__ Opnd<OP_BF16> l() const { return {__builtin_bit_cast(v4s, v2u{u[4], u[5]})}; }
    __device__ __forceinline__ v8bf mh() const { return __builtin_bit_cast(v8bf, __builtin_shufflevector(u, u, 0, 1, 2, 3)); }
    __device__ __forceinline__ v8bf hl() const { return __builtin_bit_cast(v8bf, __builtin_shufflevector(u, u, 2, 3, 4, 5)); }
};
// Six registers in a row from here on (left alone, the compiler keeps the two windows apart and copies h: two instructions a tile).
__device__ __forceinline__ void in_a_row(Split3& s) { asm("" : "+v"(s.u)); }
__device__ __forceinline__ Split3 join3(Opnd<OP_BF16> m, Opnd<OP_BF16> h, Opnd<OP_BF16> l)
{
    const v2u a = __builtin_bit_cast(v2u, m.x), b = __builtin_bit_cast(v2u, h.x), c = __builtin_bit_cast(v2u, l.x);
    Split3 s{v6u{a[0], a[1], b[0], b[1], c[0], c[1]}};
    in_a_row(s);
    return s;
}
__device__ __forceinline__ v4f minus_bf16(v4f x, Opnd<OP_BF16> y)
{
#pragma clang fp contract(off)  // (x may be a product in the caller: fused into the subtraction it would lose its rounding)
    const v2u w = __builtin_bit_cast(v2u, y.x);
#pragma unroll
    for (int r = 0; r < 4; ++r) x[r] -= __builtin_bit_cast(float, (r & 1) ? (w[r / 2] & 0xffff0000u) : (w[r / 2] << 16));
    return x;
}
__device__ __forceinline__ Split3 split3(v4f x)
{
    const Opnd<OP_BF16> h = pack<OP_BF16>(x);
    x = minus_bf16(x, h);
    const Opnd<OP_BF16> m = pack<OP_BF16>(x);
    return join3(m, h, pack<OP_BF16>(minus_bf16(x, m)));
}
// The same for values beyond the largest bf16: h is that one then, and m takes what is left.
__device__ __forceinline__ Split3 split3_any(v4f x)
{
    constexpr float MAX_BF16 = 0x1.fep127f;
    v4f c;
#pragma unroll
    for (int r = 0; r < 4; ++r) c[r] = __builtin_amdgcn_fmed3f(x[r], -MAX_BF16, MAX_BF16);
    const Opnd<OP_BF16> h = pack<OP_BF16>(c);
    x = minus_bf16(x, h);
    const Opnd<OP_BF16> m = pack<OP_BF16>(x);
    return join3(m, h, pack<OP_BF16>(minus_bf16(x, m)));
}
// acc + one part of X^T Y: the cross terms (0 and 1) or the leading term (2).  A sum of products keeps its cross terms in an
// accumulator of their own until the end: in one accumulator every term would be rounded at the size of the whole sum,
// three times per product (measured 1.5 times the error of fp32 products; with two accumulators 0.85 times).
__device__ __forceinline__ v4f tn_split(int part, Split3 x, Split3 y, v4f acc)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(part == 0 ? x.hl() : x.mh(), part == 1 ? y.hl() : y.mh(), acc, 0, 0, 0);
}

// Packed 16-bit tiles turned through LDS: a tile is written as it stands, 8 bytes a lane, column n of the matrix at row n of the patch,
// and read by the transposing read of gfx950 (ds_read_b64_tr_b16: lane n of a lane group receives element n of the four 32-byte rows
// whose pieces the group's lanes point at, a piece each).  No arithmetic, so any bits are turned; the pieces of a row are permuted by
// its group of four rows, so that neither access has a bank conflict.
constexpr int TURN16_BYTES = 512;
struct Turn16 {
    typedef __attribute__((address_space(3))) v4s* lds_v4s;
    char *put_at, *get_at;  // this lane's 8 bytes of tile 0
    __device__ __forceinline__ Turn16(float* patch, Lane ln)
    {
        const int s = ln.n >> 2;
        put_at = reinterpret_cast<char*>(patch) + 8 * (4 * ln.n + (ln.q ^ s));
        get_at = reinterpret_cast<char*>(patch) + 8 * (16 * ln.q + 4 * s + ((ln.n & 3) ^ ln.q));
    }
    __device__ __forceinline__ void put(int tile, v2u u) const { *reinterpret_cast<v2u*>(put_at + tile * TURN16_BYTES) = u; }
    __device__ __forceinline__ v2u get(int tile) const
    {
        return __builtin_bit_cast(v2u, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(get_at + tile * TURN16_BYTES)));
    }
};

// Index of lower tile (i, j), i >= j, in a packed array of NB*(NB+1)/2 tiles.
__host__ __device__ constexpr int tix(int i, int j) { return i * (i + 1) / 2 + j; }

}  // namespace triinv
