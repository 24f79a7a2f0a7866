// Residual and normalisation of one row, shared by the stand-alone kernel and the decode layer that takes the step between
// two layers into its own front end.
#pragma once
#include <math.h>

#include "common.hpp"

namespace dymoe {

// v = h + alpha * y;  out = bf16(v / rms(v)), fp32 arithmetic, by 256 threads: a thread takes 8 consecutive elements at a time
// (16-byte loads; VEC = false: one element at a time, for row lengths or pointers that rule those out), the squares are
// summed per thread, per wavefront, then over the wavefronts in order.  s_part: 4 floats of LDS.
constexpr int kNormThreads = 256;

__device__ __forceinline__ void residual_add(const uint4& h, const float4& y0, const float4& y1, float alpha, float (&v)[8])
{
    const float hv[8] = {bf16_lo(h.x), bf16_hi(h.x), bf16_lo(h.y), bf16_hi(h.y), bf16_lo(h.z), bf16_hi(h.z), bf16_lo(h.w), bf16_hi(h.w)};
    const float yv[8] = {y0.x, y0.y, y0.z, y0.w, y1.x, y1.y, y1.z, y1.w};
#pragma unroll
    for (int i = 0; i < 8; i++) v[i] = fmaf(alpha, yv[i], hv[i]);
}

template <typename YT, bool VEC>
__device__ __forceinline__ void residual_value(const uint16_t* __restrict__ hr, const YT* __restrict__ yr, float alpha, int j,
                                               float (&v)[VEC ? 8 : 1])
{
    if constexpr (VEC) {
        const uint4 h = *reinterpret_cast<const uint4*>(hr + j);
        if constexpr (sizeof(YT) == 2) {
            const uint4 y = *reinterpret_cast<const uint4*>(yr + j);
            residual_add(h, make_float4(bf16_lo(y.x), bf16_hi(y.x), bf16_lo(y.y), bf16_hi(y.y)),
                         make_float4(bf16_lo(y.z), bf16_hi(y.z), bf16_lo(y.w), bf16_hi(y.w)), alpha, v);
        } else {
            residual_add(h, *reinterpret_cast<const float4*>(yr + j), *reinterpret_cast<const float4*>(yr + j + 4), alpha, v);
        }
    } else {
        float yv;
        if constexpr (sizeof(YT) == 2) yv = bf16_bits_to_f32(yr[j]);
        else yv = yr[j];
        v[0] = fmaf(alpha, yv, bf16_bits_to_f32(hr[j]));
    }
}

template <bool VEC>
__device__ __forceinline__ void residual_square(const float (&v)[VEC ? 8 : 1], float& ss)
{
#pragma unroll
    for (int i = 0; i < (VEC ? 8 : 1); i++) ss = fmaf(v[i], v[i], ss);
}

// 1 / rms from the sums of squares of the first 256 threads (all threads of the workgroup call)
__device__ __forceinline__ float residual_inv_rms(float ss, int H, float* s_part)
{
    ss = wave_sum(ss);
    if (threadIdx.x < kNormThreads && (threadIdx.x & (kWave - 1)) == 0) s_part[threadIdx.x / kWave] = ss;
    __syncthreads();
    float tot = 0.0f;
#pragma unroll
    for (int wv = 0; wv < kNormThreads / kWave; wv++) tot += s_part[wv];
    return (tot > 0.0f) ? 1.0f / sqrtf(tot / (float)H) : 0.0f;
}

__device__ __forceinline__ uint4 residual_pack(const float (&v)[8], float inv)
{
    uint4 o;
    o.x = f32_to_bf16_bits(v[0] * inv) | (f32_to_bf16_bits(v[1] * inv) << 16);
    o.y = f32_to_bf16_bits(v[2] * inv) | (f32_to_bf16_bits(v[3] * inv) << 16);
    o.z = f32_to_bf16_bits(v[4] * inv) | (f32_to_bf16_bits(v[5] * inv) << 16);
    o.w = f32_to_bf16_bits(v[6] * inv) | (f32_to_bf16_bits(v[7] * inv) << 16);
    return o;
}

}  // namespace dymoe
