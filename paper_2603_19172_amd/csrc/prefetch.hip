// Host-resident experts: copies from pinned host memory into device buffers on
// a side stream, handed over to the compute stream through events, and the
// residual + normalisation step that chains layers of a stack.
#include <math.h>

#include "common.hpp"
#include "norm_device.hpp"

namespace dymoe {

// h_out[t,:] = bf16 of (h + alpha * y) / rms (norm_device.hpp), one workgroup per token.
template <typename YT, bool VEC>
__global__ __launch_bounds__(kNormThreads) void residual_rmsnorm_kernel(const uint16_t* __restrict__ h,
                                                                       const YT* __restrict__ y, float alpha,
                                                                       int T, int H, uint16_t* __restrict__ out)
{
    __shared__ float s_part[kNormThreads / kWave];
    const int t = blockIdx.x;
    const uint16_t* hr = h + (size_t)t * H;
    const YT* yr = y + (size_t)t * H;
    uint16_t* orow = out + (size_t)t * H;
    constexpr int W = VEC ? 8 : 1;
    float ss = 0.0f;
    for (int j = threadIdx.x * W; j < H; j += kNormThreads * W) {
        float v[W];
        residual_value<YT, VEC>(hr, yr, alpha, j, v);
        residual_square<VEC>(v, ss);
    }
    const float inv = residual_inv_rms(ss, H, s_part);
    for (int j = threadIdx.x * W; j < H; j += kNormThreads * W) {
        float v[W];
        residual_value<YT, VEC>(hr, yr, alpha, j, v);
        if constexpr (VEC) *reinterpret_cast<uint4*>(orow + j) = residual_pack(v, inv);
        else orow[j] = (uint16_t)f32_to_bf16_bits(v[0] * inv);
    }
}

}  // namespace dymoe

extern "C" {

int dymoe_prefetch_submit(dymoe_ctx* ctx, const void* host_pinned_src, void* dev_dst, size_t bytes,
                          void* side_stream, void** event_out)
{
    DYMOE_REQUIRE(event_out != nullptr);
    *event_out = nullptr;
    if (bytes > 0) DYMOE_REQUIRE(host_pinned_src != nullptr && dev_dst != nullptr);
    if (!ctx) return DYMOE_ENOCTX;
    hipStream_t st = (hipStream_t)side_stream;
    hipEvent_t ev;
    if (hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess) return DYMOE_EHIP;
    if (bytes > 0 &&
        hipMemcpyAsync(dev_dst, host_pinned_src, bytes, hipMemcpyHostToDevice, st) != hipSuccess) {
        (void)hipEventDestroy(ev);
        return DYMOE_EHIP;
    }
    if (hipEventRecord(ev, st) != hipSuccess) {
        (void)hipEventDestroy(ev);
        return DYMOE_EHIP;
    }
    *event_out = (void*)ev;
    return DYMOE_OK;
}

int dymoe_prefetch_wait(dymoe_ctx* ctx, void* event, void* compute_stream)
{
    DYMOE_REQUIRE(event != nullptr);
    if (!ctx) return DYMOE_ENOCTX;
    if (hipStreamWaitEvent((hipStream_t)compute_stream, (hipEvent_t)event, 0) != hipSuccess) return DYMOE_EHIP;
    return DYMOE_OK;
}

int dymoe_prefetch_done(dymoe_ctx* ctx, void* event)
{
    DYMOE_REQUIRE(event != nullptr);
    if (!ctx) return DYMOE_ENOCTX;
    const hipError_t r = hipEventQuery((hipEvent_t)event);
    if (r == hipSuccess) return 1;
    if (r == hipErrorNotReady) return 0;
    return DYMOE_EHIP;
}

int dymoe_prefetch_release(dymoe_ctx* ctx, void* event)
{
    DYMOE_REQUIRE(event != nullptr);
    if (!ctx) return DYMOE_ENOCTX;
    return hipEventDestroy((hipEvent_t)event) == hipSuccess ? DYMOE_OK : DYMOE_EHIP;
}

int dymoe_residual_rmsnorm(dymoe_ctx* ctx, const void* h, const void* y, int y_dtype, float alpha,
                           int T, int H, void* h_out, void* stream)
{
    DYMOE_REQUIRE(T >= 0 && H > 0);
    DYMOE_REQUIRE(y_dtype == DYMOE_OUT_BF16 || y_dtype == DYMOE_OUT_F32);
    if (T > 0) DYMOE_REQUIRE(h && y && h_out);
    if (!ctx) return DYMOE_ENOCTX;
    if (T == 0) return DYMOE_OK;
    hipStream_t st = (hipStream_t)stream;
    const bool vec = H % 8 == 0 && dymoe_aligned(h, 16) && dymoe_aligned(y, 16) && dymoe_aligned(h_out, 16);
    const dim3 grid((unsigned)T), block(dymoe::kNormThreads);
#define DYMOE_NORM(YT_, VEC_)                                                                                         \
    hipLaunchKernelGGL((dymoe::residual_rmsnorm_kernel<YT_, VEC_>), grid, block, 0, st, (const uint16_t*)h,          \
                       (const YT_*)y, alpha, T, H, (uint16_t*)h_out)
    if (y_dtype == DYMOE_OUT_BF16) {
        if (vec) DYMOE_NORM(uint16_t, true);
        else DYMOE_NORM(uint16_t, false);
    } else {
        if (vec) DYMOE_NORM(float, true);
        else DYMOE_NORM(float, false);
    }
#undef DYMOE_NORM
    DYMOE_HIP_LAUNCH_CHECK();
    return DYMOE_OK;
}

}  // extern "C"
