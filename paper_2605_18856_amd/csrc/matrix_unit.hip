// One matrix instruction on operands as they are given, for the tests of how it adds its terms: the margins of the
// filters (half_margin, kRounding) rest on that.  No part of a sweep.
#include "bsse_internal.h"
#include "mfma_device.h"

namespace bsse {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));

// One wavefront per instruction.  a, b: [count][lane][8] words, of which kinds 0 and 1 (32x32x16 in bf16 and in half
// precision) read four and kind 2 (the scaled 32x32x64 of e2m3 numbers) six; c, d: [count][lane][16];
// scales: [count][lane], the biased exponent of b's block in the lowest byte (kind 2).
__global__ void __launch_bounds__(64)
matrix_unit_kernel(int kind, const unsigned *__restrict__ a, const unsigned *__restrict__ b, const int *__restrict__ scales,
                   const float *__restrict__ c, float *__restrict__ d)
{
    const size_t lane = (size_t)blockIdx.x * 64 + threadIdx.x;
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = c[lane * 16 + r];
    const u32x4 a4 = *reinterpret_cast<const u32x4 *>(a + lane * 8), b4 = *reinterpret_cast<const u32x4 *>(b + lane * 8);
    if (kind == 0) {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a4), __builtin_bit_cast(bf16x8, b4), acc, 0, 0, 0);
    } else if (kind == 1) {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a4), __builtin_bit_cast(f16x8, b4), acc, 0, 0, 0);
    } else {
        i32x8 a6, b6;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            a6[e] = e < 6 ? (int)a[lane * 8 + e] : 0;
            b6[e] = e < 6 ? (int)b[lane * 8 + e] : 0;
        }
        acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a6, b6, acc, 2, 2, 0, 127, 0, scales[lane]);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) d[lane * 16 + r] = acc[r];
}

}  // namespace

hipError_t matrix_unit(int kind, int count, const unsigned *a, const unsigned *b, const int *scales, const float *c, float *d,
                       hipStream_t s)
{
    if (kind < 0 || kind > 2 || count < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(matrix_unit_kernel, dim3((unsigned)count), dim3(64), 0, s, kind, a, b, scales, c, d);
    return hipGetLastError();
}

}  // namespace bsse
