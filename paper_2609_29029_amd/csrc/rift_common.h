// Device-side helpers shared by the Rift kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/rift.h"

namespace rift {

typedef uint16_t bf16_t;  // bfloat16 bit pattern in memory

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf16_to_f32(bf16_t b) {
    return __uint_as_float(static_cast<uint32_t>(b) << 16);
}

// Round to nearest even; inputs are finite.
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return static_cast<bf16_t>(u >> 16);
}

// Low and high bfloat16 halves of a 32-bit word, widened exactly.
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) v += __shfl_xor(v, s);
    return v;
}

// (cos, sin) of RoPE's angle p * base^(-2j/hd), computed in float64
__device__ __forceinline__ float2 rope_entry(int p, int j, int hd, double base) {
    const double theta = pow(base, -2.0 * (double)j / (double)hd);
    const double ang = (double)p * theta;
    return make_float2((float)cos(ang), (float)sin(ang));
}

// Rotate-half RoPE of one pair, the fused forms written out: kernels that rotate
// the same row must round alike.
__device__ __forceinline__ float2 rotate_pair(float x1, float x2, float2 cs) {
    return make_float2(fmaf(x1, cs.x, -(x2 * cs.y)), fmaf(x2, cs.x, x1 * cs.y));
}

constexpr int kWave = 64;

}  // namespace rift
