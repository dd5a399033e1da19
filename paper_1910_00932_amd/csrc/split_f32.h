// fp32 products on the bf16 matrix cores, the method of Henry, Tang and Heinecke ("Leveraging the bfloat16 artificial intelligence
// datatype for higher-precision computations", 2019).  x = x0 + x1 + x2 with x0 = bf16(x), x1 = bf16(x - x0), x2 = x - x0 - x1, all
// exact (8 + 8 + 8 significant bits), and x*y is the sum of the six largest part products, each exact in fp32.  What is left out,
// x1*y2 + x2*y1 + x2*y2, is at most 2^-24 of |x*y| (the square of 0x3f807fc0, 1 + 2^-8 - 2^-17; 2.7 % of random pairs exceed 2^-26):
// one rounding of a product, where the fp32 instruction rounds sums only, and no more.  Per 32 products of a 16 x 16 tile six instructions of 16 cycles stand
// for eight of 32.  Each such group is a chain of its own, the small parts first, so that one rounding of the matrix core is of
// the size of the group's sum, and is then added in fp32: the fp32 instruction rounds the whole sum for every two products.
// Error against 64 bits, 2-norm, that instruction -> this: 1x1 and 3x3 layers of 64 to 4608 products 0.6e-7 .. 4.2e-7 ->
// 0.3e-7 .. 1.2e-7, weight gradients of 49 to 401408 pixels 0.9e-7 .. 4.1e-7 -> 0.7e-7 .. 3.9e-7 (no layer larger than before).
// Operands that the parts cannot hold (see split3), and sums that leave fp32's range where the exact one need not (x0*y0 may be
// larger than x*y), are the caller's to form again by fp32 instructions (mma_exact).
#pragma once
#include "common.h"

namespace tsm {

typedef uint32_t split_u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 split_bf16x8 __attribute__((ext_vector_type(8)));
typedef float split_f32x4 __attribute__((ext_vector_type(4)));

static constexpr int SPLIT_LOSSY = 0x093;   // class of a float: NaN (bits 0, 1), subnormal (bits 4, 7)
static constexpr uint32_t SPLIT_LEAST = (17u << 24) - 1u;   // twice the bits of 2^-110, less one: bits of zero, less one, are above it

struct Split3 { split_u32x4 p[3]; };   // eight values, three parts of them

// From 2^-110 on an operand is its three parts: its last bit is a whole multiple of 2^-133, the smallest bf16, and the matrix cores
// keep subnormal operands, products and sums.  lossy: set where x2 is subnormal, as it is for every smaller x that is not
// (below 2^-103 it may be), or NaN: an infinite x, or one that rounds to an infinite x0.  One comparison per value beside the 5.5
// instructions that cut it.
__device__ __forceinline__ Split3 split3(const float (&f)[8], bool& lossy, bool negate = false) {
    Split3 s;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float lo = negate ? -f[2 * q] : f[2 * q], hi = negate ? -f[2 * q + 1] : f[2 * q + 1];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const uint32_t w = pack_bf16x2(lo, hi);
            s.p[k][q] = w;
            if (k == 2) break;
            lo -= __uint_as_float(w << 16);
            hi -= __uint_as_float(w & 0xffff0000u);
        }
        lossy |= __builtin_amdgcn_classf(lo, SPLIT_LOSSY) || __builtin_amdgcn_classf(hi, SPLIT_LOSSY);
    }
    return s;
}

__device__ __forceinline__ Split3 split3(const float (&f)[8]) {
    bool lossy = false;
    return split3(f, lossy);
}

// sum[i][j] += a[i] * b (16 x 16 tiles, 32 products each): a chain of its own from zero, the small parts first.
template <int M>
__device__ __forceinline__ void mma_split(const Split3 (&a)[M], const Split3& b, split_f32x4 (&sum)[M]) {
    constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
    split_f32x4 t[M];
#pragma unroll
    for (int i = 0; i < M; ++i) t[i] = split_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < 6; ++k)
#pragma unroll
        for (int i = 0; i < M; ++i)
            t[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(split_bf16x8, a[i].p[PA[k]]),
                                                           __builtin_bit_cast(split_bf16x8, b.p[PB[k]]), t[i], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < M; ++i) sum[i] += t[i];
}

// The same for one a and several b: sum[j] += sign * (a * b[j]).  The matrix core's own sums lean towards minus infinity (weight
// gradients over 100352 pixels: 4.2e-7 off 64 bits, 2.0e-7 in fp32 instructions): in long sums every other chain is formed of -a
// and subtracted.  Where results are added up later instead (forward, data gradients), half of them are formed of -a: the mean over
// a tensor of sums of 2048 to 4608 products was off by 6e-8 to 8e-8 of the mean magnitude, and is by 3e-10 (6e-10).
template <int N>
__device__ __forceinline__ void mma_split_b(const Split3& a, const Split3 (&b)[N], float sign, split_f32x4 (&sum)[N]) {
    constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
    split_f32x4 t[N];
#pragma unroll
    for (int j = 0; j < N; ++j) t[j] = split_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < 6; ++k)
#pragma unroll
        for (int j = 0; j < N; ++j)
            t[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(split_bf16x8, a.p[PA[k]]),
                                                           __builtin_bit_cast(split_bf16x8, b[j].p[PB[k]]), t[j], 0, 0, 0);
#pragma unroll
    for (int j = 0; j < N; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) sum[j][r] = fmaf(t[j][r], sign, sum[j][r]);
}

// Whether a sum is infinite.  Sees no NaN: that comes with an operand that split3 reports, or of two infinite sums of opposite sign,
// which callers look for anyway (taps_inside.h).
template <int M, int N>
__device__ __forceinline__ bool split_overflow(const split_f32x4 (&sum)[M][N]) {
    float top = 0.f;
#pragma unroll
    for (int i = 0; i < M; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) top = fmaxf(top, fabsf(sum[i][j][r]));
    return top == __builtin_inff();
}

// Whether all sums are finite numbers.
template <int M, int N>
__device__ __forceinline__ bool split_finite(const split_f32x4 (&sum)[M][N]) {
    bool inf = false;
#pragma unroll
    for (int i = 0; i < M; ++i)
#pragma unroll
        for (int j = 0; j < N; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) inf |= __builtin_amdgcn_classf(sum[i][j][r], 0x207);   // NaN, infinities
    return !inf;
}

// sum[j] += 32 products by fp32 instructions, a chain of its own: a(j, e) and b(j, e) are the eight values that a lane supplies to
// split3.  For the rare operands that cannot be cut, so with few registers.
template <int N, typename A, typename B>
__device__ __forceinline__ void mma_exact(A a, B b, split_f32x4 (&sum)[N]) {
    split_f32x4 t[N];
#pragma unroll
    for (int j = 0; j < N; ++j) t[j] = split_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int j = 0; j < N; ++j) t[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a(j, e), b(j, e), t[j], 0, 0, 0);
#pragma unroll
    for (int j = 0; j < N; ++j) sum[j] += t[j];
}

}  // namespace tsm
