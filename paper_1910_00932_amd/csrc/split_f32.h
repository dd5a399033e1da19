// fp32 products on the bf16 matrix cores.  x = x0 + x1 + x2 with x0 = bf16(x), x1 = bf16(x - x0), x2 = x - x0 - x1, all exact
// (8 + 8 + 8 significant bits), and x*y is the sum of the six products of order 2^-18 and above, each exact in fp32; what is
// left out, x1*y2 + x2*y1 + x2*y2, is at most 2^-26 of |x*y|.  Per 32 products of a 16 x 16 tile six instructions of 16 cycles stand
// for eight of 32.  Each such group is a chain of its own, the small parts first, so that one rounding of the matrix core is of
// the size of the group's sum, and is then added in fp32: the fp32 instruction rounds the whole sum for every two products.
// Error against 64 bits, 2-norm, that instruction -> this: 1x1 and 3x3 layers of 64 to 4608 products 0.6e-7 .. 4.2e-7 ->
// 0.3e-7 .. 1.2e-7, weight gradients of 49 to 401408 pixels 0.9e-7 .. 4.1e-7 -> 0.7e-7 .. 3.9e-7 (no layer larger than before).
// An infinite operand, or one that rounds to an infinite x0, makes NaN of its sums (x - x0): callers form those again.
// Operands and products below 2^-108 lose the bits that bf16 and fp32 cannot hold.
#pragma once
#include "common.h"

namespace tsm {

typedef uint32_t split_u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 split_bf16x8 __attribute__((ext_vector_type(8)));
typedef float split_f32x4 __attribute__((ext_vector_type(4)));

struct Split3 { split_u32x4 p[3]; };   // eight values, three parts of them

__device__ __forceinline__ Split3 split3(const float (&f)[8]) {
    Split3 s;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float lo = f[2 * q], hi = f[2 * q + 1];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const uint32_t w = pack_bf16x2(lo, hi);
            s.p[k][q] = w;
            lo -= __uint_as_float(w << 16);
            hi -= __uint_as_float(w & 0xffff0000u);
        }
    }
    return s;
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

// The same for one a and several b: sum[j] += sign * (a * b[j]).  The matrix core's own sums lean towards minus infinity
// (weight gradients over 100352 pixels: 4.2e-7 off 64 bits, 2.0e-7 in fp32 instructions): in long sums every other
// chain is formed of -a and subtracted.
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

}  // namespace tsm
