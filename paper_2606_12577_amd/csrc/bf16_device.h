// 16x16 block products on the matrix cores: operand types, the BF16 pair of an
// FP32 vector and the layout constants of the block-row records.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace cs {
namespace {

constexpr int META_COLS = 5;   // block columns that a row record holds
typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ unsigned short f2bf(float f) {   // round to nearest even
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (unsigned short)(u >> 16);
}
__device__ __forceinline__ float bf2f(unsigned short h) { return __uint_as_float((uint32_t)h << 16); }

// v = hi + lo, both rounded to nearest even: gfx950 converts two floats per
// instruction (three instructions per element; the integer form of f2bf took
// ten, which bound the sweeps of many rows per CU).
__device__ __forceinline__ void split(const float (&v)[4], bf16x4 &hi, bf16x4 &lo) {
    typedef float f32v4 __attribute__((ext_vector_type(4)));
    typedef __bf16 bfv4 __attribute__((ext_vector_type(4)));
    const f32v4 f = {v[0], v[1], v[2], v[3]};
    hi = __builtin_bit_cast(bf16x4, __builtin_convertvector(f, bfv4));
    f32v4 d;
#pragma unroll
    for (int t = 0; t < 4; ++t) d[t] = f[t] - bf2f((unsigned short)hi[t]);
    lo = __builtin_bit_cast(bf16x4, __builtin_convertvector(d, bfv4));
}

__device__ __forceinline__ f32x4 mfma(bf16x4 a, bf16x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

}  // namespace
}  // namespace cs
