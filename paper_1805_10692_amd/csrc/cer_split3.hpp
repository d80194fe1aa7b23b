// fp32 numbers as sums of bf16 numbers, for the bf16 matrix cores (gfx950).
//
// A binary32 significand has 24 bits, a bf16 one has 8: x = p0 + p1 + p2 with p0 = bf16(x), p1 = bf16(x - p0),
// p2 = x - p0 - p1 is exact (both differences are exact in binary32, the last one fits 8 bits), for |x| from 2^-110 up to the
// largest number that rounds to a finite bf16 one.  Other numbers have no such pieces -- those below lose what lies under
// 2^-133, the smallest bf16 number -- and a product that meets them (below 2^-110: in which that shows) is formed in binary32.
//
// Products of two pieces are exact in binary32 and the matrix cores add them up in binary32, so a contraction over pieces has
// the inputs and the accumulation of the fp32 one.  With two pieces of the weight one of its six products is left out, with
// three pieces three of nine: together below 2^-25 of the product, half a unit of what rounding a binary32 product costs.
// Against fp64 the sums come closer than with the fp32 matrix instructions (2-norm; X normal, and the same cut at 0):
//                        one piece             two                   three                 fp32 instruction
//   512 x 4608           1.3e-7  4.9e-8        7.3e-8  4.3e-8        8.9e-8  7.6e-8        2.3e-7  1.5e-7 - 5.6e-8
//   700 x 1200           1.2e-7  5.4e-8        6.1e-8  4.3e-8        7.4e-8  6.3e-8        1.6e-7  1.2e-7 - 5.5e-8
//   256 x 25088          1.6e-7  6.4e-8        1.1e-7  6.5e-8        1.2e-7  8.7e-8        3.6e-7  1.8e-7 - 6.7e-8
// The bf16 matrix instructions run at 16 times the rate of the fp32 ones: three products (one piece), five or six cost a fifth
// to three eighths of the fp32 instruction's time.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "cer_internal.hpp"

namespace cer {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

// Forms of the decoded weights: one to three pieces, or kUniform (two numbers, see uniform_pieces).
constexpr int kUniform = 4;
__host__ __device__ constexpr int weight_planes(int form) { return form == kUniform ? 2 : form; }

__device__ __forceinline__ uint32_t bf16_pair(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{lo, hi}, bf16x2));
}

// Pieces of a pair of numbers that are finite and round to finite bf16 numbers; the return value is a NaN for other numbers,
// and else the size of the third pieces: 0 where the first two are all there is.
__device__ __forceinline__ float split3_pair(float a, float b, uint32_t p[3]) {
    p[0] = bf16_pair(a, b);
    const float ra = a - __uint_as_float(p[0] << 16), rb = b - __uint_as_float(p[0] & 0xFFFF0000u);
    p[1] = bf16_pair(ra, rb);
    const float qa = ra - __uint_as_float(p[1] << 16), qb = rb - __uint_as_float(p[1] & 0xFFFF0000u);
    p[2] = bf16_pair(qa, qb);
    return fabsf(qa) + fabsf(qb);
}

// A number with bits that the pieces may not reach: 0 < |x| < 2^-110.
__device__ __forceinline__ bool split_lossy(float x) { return (__float_as_uint(x) << 1) - 1u < 2u * 0x08800000u - 1u; }

// Pieces of one finite number; numbers that would round to infinity are cut instead.
__device__ __forceinline__ void split3_finite(float x, uint32_t p[3]) {
    const uint32_t u = __float_as_uint(x);
    p[0] = (u & 0x7FFFFFFFu) >= 0x7F7F0000u ? u >> 16 : bf16_pair(x, 0.f) & 0xFFFFu;
    const float r = x - __uint_as_float(p[0] << 16);
    p[1] = bf16_pair(r, 0.f) & 0xFFFFu;
    p[2] = bf16_pair(r - __uint_as_float(p[1] << 16), 0.f) & 0xFFFFu;
}

// Eight numbers -> three times eight bf16, in the order given; the return value is that of split3_pair, added up.
__device__ __forceinline__ float split3_8(const float x[8], uint4 out[3]) {
    uint32_t w[3][4];
    float odd = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t p[3];
        odd += split3_pair(x[2 * i], x[2 * i + 1], p);
#pragma unroll
        for (int j = 0; j < 3; ++j) w[j][i] = p[j];
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) out[j] = make_uint4(w[j][0], w[j][1], w[j][2], w[j][3]);
    return odd;
}

__device__ __forceinline__ floatx16 mfma_bf16(uint4 a, uint4 b, floatx16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// The products of PW pieces of one factor with three of the other that reach 2^-25 of the result.  PW > 1: all but the largest
// are added up apart, in lo -- every matrix instruction rounds the sum it adds to, and in one sum the four or five small
// products rounded it as often as the large one: errors of 2.3e-7 against 1.6e-7 with binary32 products (700 x 1200, 2-norm).
// kForm: the number of pieces, or kUniform.
template <int kForm>
__device__ __forceinline__ void mfma_pieces(const uint4* a, const uint4* b, floatx16& hi, floatx16& lo) {
    constexpr int kPlanes = weight_planes(kForm);
#pragma unroll
    for (int s = 2; s >= 0; --s)
#pragma unroll
        for (int i = 0; i < kPlanes; ++i)
            if (s - i >= 0 && !(kForm == kUniform && i == 1 && s == 2)) {
                floatx16& c = kPlanes > 1 && s > 0 ? lo : hi;
                c = mfma_bf16(a[i], b[s - i], c);
            }
}

// Weights on a uniform grid through zero (uniform_grid in cer_capi.cpp): w = scale . (unit . j + e) with an integer j of at most eight
// bits, one bf16 number with the power of two, and what the rounding of the grid's points leaves, |scale . e| <= 2^-22 |w|, as another
// one.  The product of e needs X's first piece only, so that there are four products instead of six.  What is left out -- e's own
// rounding, and its products with the further pieces of X -- is below 2^-29 of the product (2^-25 with three pieces).  1 <= scale < 2:
// the products are no larger than with w itself.  Errors against fp64 are two thirds of three pieces' in the mean (uniform_grid):
// scale . hi + scale . lo is rounded once, and of the five small products one is left that matters.
__device__ __forceinline__ uint32_t uniform_pieces(float w, const UniformGrid& g) {
    const double j = rint((double)w * g.inverse), step = (double)g.scale * (double)g.unit;
    return bf16_pair((float)j * g.unit, (float)(fma(-j, step, (double)w) * g.inverse) * g.unit);
}

// X from row `row` on, as a buffer that ends with row `end` - 1: loads behind it return zero.  The range check of a buffer load
// covers its vector offset only, so the row goes into the base address (scalar arithmetic) and not into the scalar offset.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t x_rows(const float* X, uint32_t L, uint32_t row, uint32_t end) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(X + (size_t)row * L), 0, row < end ? (end - row) * L * 4u : 0u, 0x00020000);
}

}  // namespace cer
