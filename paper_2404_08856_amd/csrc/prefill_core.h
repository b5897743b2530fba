// Operand layouts of the prompt kernels.
//
// Weights: the packed 1 KiB blocks of common.h, unchanged (A operand).  Activations X[R, K]: every value as a sum of T
// 16-bit terms, each an operand of its own -- 16 rows fill the 16 columns of the B operand -- and the T products go into the
// same sum: no column of a tile is unused and no sum over term columns is needed.  Block (row tile rt of 16 rows, K-step s,
// term t) is the 1 KiB at index (rt * KS + s) * T + t, lane l = r + 16 g holding X[16 rt + r][32 s + 8 g .. + 7].
//
//  T = 3  bf16 terms, as everywhere else.
//  T = 2  f16 terms of the values times a power of two per (row, block of 128 or 64 columns), chosen by whoever writes the
//         block so that its largest magnitude is in [2^14, 2^15); the inverse factors are an array next to X.  2/3 of the matrix work.
#pragma once
#include "common.h"
#include "launch.h"

namespace spd {

template <int T>
__device__ __forceinline__ size_t ppack_index(int row, int k, int KS, int t) {       // element offset (16-bit units) of X[row][k] term t
    return (((size_t)(row >> 4) * KS + (k >> 5)) * T + t) * 512 + packed_elem_index(row & 15, k & 31);
}
// place of the inverse factor of (row, block of columns), n_blocks blocks per row
__device__ __forceinline__ size_t pscale_index(int row, int block, int n_blocks) { return ((size_t)(row >> 4) * n_blocks + block) * 16 + (row & 15); }

// Powers of two: 2^k with 2^k * m in [2^14, 2^15) for the largest magnitude m of a block, and 2^-k.  A block of zeros or
// with an infinite value stays as it is; k <= 126, so that both are ordinary numbers.
__device__ __forceinline__ float block_factor(float m) {
    const int e = (int)(__float_as_uint(m) >> 23);                       // m >= 0
    return __uint_as_float((uint32_t)(127 + (e == 255 || m == 0.f ? 0 : min(141 - e, 126))) << 23);
}
__device__ __forceinline__ float power_inverse(float p) { return __uint_as_float(0x7f000000u - __float_as_uint(p)); }

// Two products a b and c d, times a block's factor, -> their f16 terms, term t of both packed in one register (the first in the
// low half).  The second term is the rest of the exact product: what reaches the matrix cores has been rounded once, at 22 to 23 bits, and not twice.
__device__ __forceinline__ void split2_products(float a, float b, float c, float d, float factor, float inverse, uint32_t (&t)[2]) {
    typedef __attribute__((ext_vector_type(2))) float f32x2_t;
    typedef __attribute__((ext_vector_type(2))) _Float16 f16x2_t;
    const f16x2_t hi = __builtin_convertvector((f32x2_t{a * b * factor, c * d * factor}), f16x2_t);
    const float ra = __builtin_fmaf(a, b, -(float)hi.x * inverse), rc = __builtin_fmaf(c, d, -(float)hi.y * inverse);
    t[0] = __builtin_bit_cast(uint32_t, hi);
    t[1] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t{ra * factor, rc * factor}), f16x2_t));
}
// four consecutive values x[i] y[i] (k % 4 == 0) of one row into the packed layout, 8 bytes per term (T = 3: the factor is not used)
template <int T>
__device__ __forceinline__ void ppack_store4(uint16_t *X, int row, int k, int KS, const float (&x)[4], const float (&y)[4], float factor) {
    uint32_t lo[T], hi[T];
    if constexpr (T == 2) {
        const float inverse = power_inverse(factor);
        split2_products(x[0], y[0], x[1], y[1], factor, inverse, lo);
        split2_products(x[2], y[2], x[3], y[3], factor, inverse, hi);
    } else {
        split3_pair(x[0] * y[0], x[1] * y[1], lo);
        split3_pair(x[2] * y[2], x[3] * y[3], hi);
    }
#pragma unroll
    for (int t = 0; t < T; ++t) *reinterpret_cast<uint2 *>(X + ppack_index<T>(row, k, KS, t)) = uint2{lo[t], hi[t]};
}

}  // namespace spd
