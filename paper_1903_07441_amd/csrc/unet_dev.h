// Device helpers shared by the network's kernels (unet.hip, conv3.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace twg {
namespace ndev {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// ---- bf16 helpers -------------------------------------------------------
__device__ __forceinline__ float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
// round to nearest even, two at once in one instruction; NaN stays a quiet NaN
__device__ __forceinline__ uint32_t pack2(float lo, float hi)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}
// ReLU that keeps a NaN a NaN (the hardware max would turn it into 0), so a
// broken parameter shows up in the network's output
__device__ __forceinline__ float relu(float v) { return v != v ? v : fmaxf(v, 0.f); }
__device__ __forceinline__ bool bf_pos(uint32_t h) { return (h & 0x8000u) == 0 && (h & 0x7fffu) != 0; }

__device__ __forceinline__ bf16x8 as_bf8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }

__device__ __forceinline__ void unpack8(uint4 v, float *f)
{
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f[2 * i] = bf_lo(w[i]);
        f[2 * i + 1] = bf_hi(w[i]);
    }
}
__device__ __forceinline__ uint4 pack8(const float *f)
{
    return make_uint4(pack2(f[0], f[1]), pack2(f[2], f[3]), pack2(f[4], f[5]), pack2(f[6], f[7]));
}

// the mean of a 2x2 block of pixels, 8 channels each, rounded to bf16
__device__ __forceinline__ uint4 mean4(uint4 v00, uint4 v01, uint4 v10, uint4 v11)
{
    float a[8], t[8], s[8];
    unpack8(v00, a);
    unpack8(v01, t);
#pragma unroll
    for (int i = 0; i < 8; ++i) s[i] = a[i] + t[i];
    unpack8(v10, a);
    unpack8(v11, t);
#pragma unroll
    for (int i = 0; i < 8; ++i) s[i] = (s[i] + (a[i] + t[i])) * 0.25f;
    return pack8(s);
}

// y = hb + sum_c hw[c] d[c] for a pixel's 32 channels v (FP32, channel
// order); d receives the channels
__device__ __forceinline__ float head_value(const uint4 (&v)[4], const float *__restrict__ hw, float hb, float *d)
{
#pragma unroll
    for (int q = 0; q < 4; ++q) unpack8(v[q], d + 8 * q);
    float y = hb;
#pragma unroll
    for (int c = 0; c < 32; ++c) y = y + hw[c] * d[c];
    return y;
}

}  // namespace ndev
}  // namespace twg
