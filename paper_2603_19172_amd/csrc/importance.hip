// Expert importance (heavy-hitter token load / gate score) and the
// importance-ranked bit-width assignment.  Both are tiny: integer histograms
// and an E x E ranking, sized for one or a few workgroups.
#include <math.h>

#include <type_traits>

#include "common.hpp"
#include "assign.hpp"

namespace dymoe {

constexpr int kImpThreads = 1024;

// zero-fill without hipMemsetAsync (the calls may be captured into a graph)
__global__ void zero_i32_kernel(int32_t* a, int32_t* b, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        a[i] = 0;
        b[i] = 0;
    }
}

// Prefill: a token is a heavy hitter when fewer than k_hh tokens precede it in
// the order (score descending, token index ascending).  kImpLanes adjacent
// lanes share one token: all T scores pass through LDS, 2048 per trip (a
// thread's two requested together), each lane compares the token against its
// share of every 1024 of them (four scores per read), and the partial counts
// are added across the lanes.  (32 lanes per token and 1024 threads: with 8
// lanes and 256 threads the 2048 tokens of the 128-expert layer kept 256
// wavefronts busy on a chip of 1024 SIMDs, a memory latency per 256 scores,
// and four times as many workgroups queued up at the E global counters.)  The token's first lane
// then adds its k routed experts to the workgroup's LDS histograms (load and,
// if heavy, importance); the workgroup adds its non-zero bins to the global
// ones, which the caller has zeroed.
constexpr int kImpLanes = 32;
constexpr int kImpTokens = kImpThreads / kImpLanes;      // tokens per workgroup
constexpr int kImpStage = 2 * kImpThreads;               // scores in LDS per trip

__global__ __launch_bounds__(kImpThreads) void importance_prefill_kernel(
    const int32_t* __restrict__ idx, const float* __restrict__ score, int T, int E, int k, int k_hh,
    int32_t* __restrict__ importance, int32_t* __restrict__ load)
{
    __shared__ __attribute__((aligned(16))) float tile[kImpStage];
    __shared__ int32_t s_load[DYMOE_MAX_EXPERTS];
    __shared__ int32_t s_imp[DYMOE_MAX_EXPERTS];
    for (int e = threadIdx.x; e < E; e += kImpThreads) {
        s_load[e] = 0;
        s_imp[e] = 0;
    }
    const int part = threadIdx.x % kImpLanes;
    const int t = blockIdx.x * kImpTokens + threadIdx.x / kImpLanes;
    const float mine = (t < T) ? score[t] : 0.0f;
    int before = 0;
    constexpr int kSpan = kImpThreads / kImpLanes;     // scores of a tile that one lane looks at
    for (int base = 0; base < T; base += kImpStage) {
        // a thread's eight scores of this trip are requested together (one at a time, every 256 scores cost a
        // memory latency: eight of them for the 2048 tokens of the 128-expert layer)
        float v[kImpStage / kImpThreads];
#pragma unroll
        for (int u = 0; u < kImpStage / kImpThreads; u++) {
            const int i = base + u * kImpThreads + (int)threadIdx.x;
            // slots past the end hold -inf at an index past every token: never counted
            v[u] = (i < T) ? score[i] : -INFINITY;
        }
        __syncthreads();                               // the previous trip's scores have been read
#pragma unroll
        for (int u = 0; u < kImpStage / kImpThreads; u++) tile[u * kImpThreads + threadIdx.x] = v[u];
        __syncthreads();
        const int pieces = min(kImpStage / kImpThreads, (T - base + kImpThreads - 1) / kImpThreads);
        for (int piece = 0; piece < pieces; piece++) {
#pragma unroll
            for (int j = part * kSpan; j < (part + 1) * kSpan; j += 4) {
                const float4 s4 = *reinterpret_cast<const float4*>(tile + piece * kImpThreads + j);
                const int u0 = base + piece * kImpThreads + j;
                before += (s4.x > mine || (s4.x == mine && u0 + 0 < t)) ? 1 : 0;
                before += (s4.y > mine || (s4.y == mine && u0 + 1 < t)) ? 1 : 0;
                before += (s4.z > mine || (s4.z == mine && u0 + 2 < t)) ? 1 : 0;
                before += (s4.w > mine || (s4.w == mine && u0 + 3 < t)) ? 1 : 0;
            }
        }
    }
#pragma unroll
    for (int o = 1; o < kImpLanes; o <<= 1) before += __shfl_xor(before, o, kWave);
    const bool heavy = (t < T) && before < k_hh;
    if (t < T && part == 0) {
        for (int s = 0; s < k; s++) {
            const int e = idx[(size_t)t * k + s];
            if (e < 0 || e >= E) continue;
            atomicAdd(&s_load[e], 1);
            if (heavy) atomicAdd(&s_imp[e], 1);
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += kImpThreads) {
        if (s_load[e]) atomicAdd(&load[e], s_load[e]);
        if (s_imp[e]) atomicAdd(&importance[e], s_imp[e]);
    }
}

// Both phases in one workgroup and one launch: histograms live in LDS, so there is nothing to zero beforehand, and the
// assignment can follow on the spot.
//   prefill  up to 256 tokens: as many lanes per token as 1024 threads give (at least four) share its comparisons with the
//            T scores, which are the caller's or, x given, the row norms of x (token_norm_kernel's arithmetic; stored to
//            score as well)
//   decode   any number of tokens: a thread adds up its expert's probabilities in token order, more than eight tokens of
//            fewer than 768 experts through LDS, 8192 at a time
// Bound: latency of two or three dependent trips to memory.  61 tokens x 128 experts, decode: 5 us with the assignment,
// where zero-fill, load histogram, the sum with a thread walking the tokens in memory and the assignment took 4 + 4.4 +
// 15 + 4.8 us; 16 tokens, prefill: 4 us with norms and assignment for 2.1 + 4 + 2.4.  The comparisons grow with the square of
// the tokens and only one compute unit makes them: 19 us at 512 tokens, where importance_prefill_kernel and the assignment
// take 5.5 + 5.
constexpr int kImpBlock = 1024;
constexpr int kImpBlockTokens = 256;                     // prefill
constexpr int kImpNormBytes = 64 << 10;                  // x up to this size and ...
constexpr int kImpNormTokens = 64;                       // ... this many rows: its norms are taken here as well
constexpr int kImpProbs = 8192;

template <bool PREFILL, bool ASSIGN>
__global__ __launch_bounds__(kImpBlock) void importance_block_kernel(
    const uint16_t* __restrict__ x, int H, const int32_t* __restrict__ idx, float* __restrict__ score,
    const float* __restrict__ probs, int T, int E, int k, int k_hh, void* __restrict__ importance, int32_t* __restrict__ load,
    TierTable tiers, int floor_bits, uint8_t* __restrict__ bits, int32_t* __restrict__ rank)
{
    using ImpT = typename std::conditional<PREFILL, int32_t, float>::type;
    __shared__ int32_t s_load[DYMOE_MAX_EXPERTS];
    __shared__ ImpT s_imp[DYMOE_MAX_EXPERTS];
    __shared__ __attribute__((aligned(16))) float s_buf[PREFILL ? kImpBlockTokens : kImpProbs];
    const int tid = threadIdx.x;
    for (int e = tid; e < E; e += kImpBlock) {
        s_load[e] = 0;
        s_imp[e] = 0;
    }
    if constexpr (PREFILL) {
        if (x) {
            const int lane = tid & (kWave - 1);
            for (int t = tid / kWave; t < T; t += kImpBlock / kWave) {
                const float n = token_norm(x + (size_t)t * H, H, lane);
                if (lane == 0) {
                    score[t] = n;
                    s_buf[t] = n;
                }
            }
        } else if (tid < T) {
            s_buf[tid] = score[tid];
        }
        if (tid >= T && tid < kImpBlockTokens) s_buf[tid] = -INFINITY;      // past every token: never counted
        __syncthreads();
        int lanes = 64;
        while (lanes * T > kImpBlock) lanes >>= 1;
        const int t = tid / lanes, part = tid % lanes;
        int before = 0;
        if (t < T) {
            const float mine = s_buf[t];
            for (int j = 4 * part; j < T; j += 4 * lanes) {
                const float4 s4 = *reinterpret_cast<const float4*>(s_buf + j);
                before += (s4.x > mine || (s4.x == mine && j + 0 < t)) ? 1 : 0;
                before += (s4.y > mine || (s4.y == mine && j + 1 < t)) ? 1 : 0;
                before += (s4.z > mine || (s4.z == mine && j + 2 < t)) ? 1 : 0;
                before += (s4.w > mine || (s4.w == mine && j + 3 < t)) ? 1 : 0;
            }
        }
        for (int o = 1; o < lanes; o <<= 1) before += __shfl_xor(before, o, kWave);
        if (t < T)
            for (int s = part; s < k; s += lanes) {
                const int e = idx[(size_t)t * k + s];
                if (e < 0 || e >= E) continue;
                atomicAdd(&s_load[e], 1);
                if (before < k_hh) atomicAdd(&s_imp[e], 1);
            }
    } else {
        __syncthreads();
        const long pairs = (long)T * k;
        for (long p = tid; p < pairs; p += kImpBlock) {
            const int e = idx[p];
            if (e >= 0 && e < E) atomicAdd(&s_load[e], 1);
        }
        float g = 0.0f;                                                     // of expert tid
        const int step = kImpProbs / E;
        // A batch of at most eight tokens is one trip to memory either way, and staging adds two barriers to it; from 768
        // experts on the experts' own threads have as much in flight as the whole workgroup.  Straight from memory / staged,
        // us: 1 token x 8 experts 2.0 / 2.4, 8 x 768 2.4 / 2.7, 1024 x 768 65 / 73, but 1024 x 513 64 / 59.
        if (T == 1) {
            if (tid < E) g += probs[tid];
        } else if (T <= 8 || E >= 768) {
            if (tid < E)
                for (int t0 = 0; t0 < T; t0 += 8) {
                    float v[8];
#pragma unroll
                    for (int u = 0; u < 8; u++) v[u] = probs[(size_t)min(t0 + u, T - 1) * E + tid];
#pragma unroll
                    for (int u = 0; u < 8; u++)
                        if (t0 + u < T) g += v[u];
                }
        } else {
            for (int t0 = 0; t0 < T; t0 += step) {
                const int n = min(step, T - t0);
                float v[kImpProbs / kImpBlock];
#pragma unroll
                for (int u = 0; u < kImpProbs / kImpBlock; u++) {
                    const int i = u * kImpBlock + tid;
                    v[u] = (i < n * E) ? probs[(size_t)t0 * E + i] : 0.0f;
                }
                __syncthreads();                                            // the previous trip's have been read
#pragma unroll
                for (int u = 0; u < kImpProbs / kImpBlock; u++) s_buf[u * kImpBlock + tid] = v[u];
                __syncthreads();
                if (tid < E)
#pragma unroll 8
                    for (int t = 0; t < n; t++) g += s_buf[t * E + tid];
            }
        }
        if (tid < E) s_imp[tid] = (T <= 1) ? g : g / (float)T;
    }
    __syncthreads();
    for (int e = tid; e < E; e += kImpBlock) {
        load[e] = s_load[e];
        reinterpret_cast<ImpT*>(importance)[e] = s_imp[e];
    }
    if constexpr (ASSIGN) assign_all<ImpT>(kImpBlock, E, s_imp, s_load, tiers, floor_bits, bits, rank);
}

// Row norms, and zeros where the importance kernel behind it adds up.
__global__ __launch_bounds__(256) void norm_and_zero_kernel(const uint16_t* __restrict__ x, int T, int H, float* __restrict__ score,
                                                            int32_t* __restrict__ importance, int32_t* __restrict__ load, int E)
{
    if (blockIdx.x == 0) {
        for (int e = threadIdx.x; e < E; e += 256) {
            importance[e] = 0;
            load[e] = 0;
        }
    }
    const int t = blockIdx.x * (256 / kWave) + threadIdx.x / kWave;
    if (t >= T) return;
    const int lane = threadIdx.x & (kWave - 1);
    const float n = token_norm(x + (size_t)t * H, H, lane);
    if (lane == 0) score[t] = n;
}

// One workgroup of 1024 threads: up to eight lanes share an expert's ranking.
template <typename ImpT>
__global__ __launch_bounds__(DYMOE_MAX_EXPERTS) void assign_precision_kernel(
    const ImpT* __restrict__ importance, const int32_t* __restrict__ load, int E, TierTable tiers,
    int floor_bits, uint8_t* __restrict__ bits, int32_t* __restrict__ rank)
{
    __shared__ ImpT s_imp[DYMOE_MAX_EXPERTS];
    __shared__ int32_t s_load[DYMOE_MAX_EXPERTS];
    for (int e = threadIdx.x; e < E; e += blockDim.x) {
        s_imp[e] = importance[e];
        s_load[e] = load ? load[e] : 0;
    }
    __syncthreads();
    assign_all<ImpT>((int)blockDim.x, E, s_imp, s_load, tiers, floor_bits, bits, rank);
}

}  // namespace dymoe

extern "C" {

int dymoe_expert_importance(dymoe_ctx* ctx, int phase, const int32_t* idx, const float* probs,
                            const float* token_score, int T, int E, int k, int k_hh,
                            void* importance, int32_t* load, void* stream)
{
    DYMOE_REQUIRE(importance && load);
    DYMOE_REQUIRE(phase == DYMOE_PHASE_PREFILL || phase == DYMOE_PHASE_DECODE);
    DYMOE_REQUIRE(T >= 0 && E > 0 && k > 0 && k <= E);
    if (phase == DYMOE_PHASE_PREFILL) DYMOE_REQUIRE(k_hh >= 0 && k_hh <= T);
    if (T > 0) {
        DYMOE_REQUIRE(idx != nullptr);
        if (phase == DYMOE_PHASE_PREFILL) DYMOE_REQUIRE(token_score != nullptr);
        else DYMOE_REQUIRE(probs != nullptr);
    }
    if (E > DYMOE_MAX_EXPERTS) return DYMOE_ENOTSUP;
    if (!ctx) return DYMOE_ENOCTX;
    hipStream_t st = (hipStream_t)stream;
    const bool prefill = phase == DYMOE_PHASE_PREFILL;
    const dymoe::TierTable none = {};
    if (!prefill) {
        dymoe_launch(ctx, DYMOE_K_IMPORTANCE, (dymoe::importance_block_kernel<false, false>), dim3(1), dim3(dymoe::kImpBlock), 0, st,
                     nullptr, 0, idx, nullptr, probs, T, E, k, 0, importance, load, none, 0, nullptr, nullptr);
    } else if (T <= dymoe::kImpBlockTokens) {
        // (const: without x the scores are only read)
        dymoe_launch(ctx, DYMOE_K_IMPORTANCE, (dymoe::importance_block_kernel<true, false>), dim3(1), dim3(dymoe::kImpBlock), 0, st,
                     nullptr, 0, idx, const_cast<float*>(token_score), nullptr, T, E, k, k_hh, importance, load, none, 0, nullptr,
                     nullptr);
    } else {
        hipLaunchKernelGGL(dymoe::zero_i32_kernel, dim3((E + 255) / 256), dim3(256), 0, st, load, (int32_t*)importance, E);
        DYMOE_HIP_LAUNCH_CHECK();
        dymoe_launch(ctx, DYMOE_K_IMPORTANCE, dymoe::importance_prefill_kernel,
                     dim3((unsigned)((T + dymoe::kImpTokens - 1) / dymoe::kImpTokens)), dim3(dymoe::kImpThreads), 0, st, idx,
                     token_score, T, E, k, k_hh, (int32_t*)importance, load);
    }
    DYMOE_HIP_LAUNCH_CHECK();
    return DYMOE_OK;
}

int dymoe_rank_experts(dymoe_ctx* ctx, int phase, const void* x, int H, const int32_t* idx, const float* probs, float* token_score,
                       int T, int E, int k, int k_hh, int n_tiers, const int32_t* tier_count, const uint8_t* tier_bits,
                       int floor_bits, void* importance, int32_t* load, uint8_t* bits, int32_t* rank, void* stream)
{
    DYMOE_REQUIRE(importance && load && bits && rank);
    DYMOE_REQUIRE(phase == DYMOE_PHASE_PREFILL || phase == DYMOE_PHASE_DECODE);
    DYMOE_REQUIRE(T >= 0 && E > 0 && k > 0 && k <= E);
    DYMOE_REQUIRE(floor_bits == 0 || floor_bits == 2 || floor_bits == 4 || floor_bits == 8 || floor_bits == 16);
    const bool prefill = phase == DYMOE_PHASE_PREFILL;
    if (prefill) DYMOE_REQUIRE(k_hh >= 0 && k_hh <= T);
    if (prefill && x) DYMOE_REQUIRE(H > 0 && H % 8 == 0 && dymoe_aligned(x, 16));
    if (T > 0) {
        DYMOE_REQUIRE(idx != nullptr);
        if (prefill) DYMOE_REQUIRE(token_score != nullptr);
        else DYMOE_REQUIRE(probs != nullptr);
    }
    dymoe::TierTable tt;
    DYMOE_REQUIRE(dymoe::make_tier_table(E, n_tiers, tier_count, tier_bits, tt) == DYMOE_OK);
    if (E > DYMOE_MAX_EXPERTS) return DYMOE_ENOTSUP;
    if (!ctx) return DYMOE_ENOCTX;
    hipStream_t st = (hipStream_t)stream;
    const uint16_t* xb = (const uint16_t*)x;
    if (!prefill) {
        dymoe_launch(ctx, DYMOE_K_IMPORTANCE, (dymoe::importance_block_kernel<false, true>), dim3(1), dim3(dymoe::kImpBlock), 0, st,
                     nullptr, 0, idx, nullptr, probs, T, E, k, 0, importance, load, tt, floor_bits, bits, rank);
        DYMOE_HIP_LAUNCH_CHECK();
        return DYMOE_OK;
    }
    if (T <= dymoe::kImpBlockTokens) {
        // One workgroup does not read more than 64 KiB of x in the time of a launch, nor, however short the rows, more than
        // four after the other by each of its 16 wavefronts: beyond, the norms have a launch of their own.  Inside / outside,
        // us: 64 x 128 5.1 / 5.2, 80 x 128 5.7 / 5.4, 256 x 128 13.3 / 7.9, 64 x 512 5.1 / 5.3 (8 experts).
        const bool inside = x && T <= dymoe::kImpNormTokens && (size_t)T * H * 2 <= (size_t)dymoe::kImpNormBytes;
        if (x && !inside && T > 0) {
            const int rc = dymoe_token_score_norm(ctx, x, T, H, token_score, stream);
            if (rc != DYMOE_OK) return rc;
        }
        dymoe_launch(ctx, DYMOE_K_IMPORTANCE, (dymoe::importance_block_kernel<true, true>), dim3(1), dim3(dymoe::kImpBlock), 0, st,
                     inside ? xb : nullptr, H, idx, token_score, nullptr, T, E, k, k_hh, importance, load, tt, floor_bits, bits, rank);
        DYMOE_HIP_LAUNCH_CHECK();
        return DYMOE_OK;
    }
    if (!x) {
        const int rc = dymoe_expert_importance(ctx, phase, idx, probs, token_score, T, E, k, k_hh, importance, load, stream);
        return rc != DYMOE_OK ? rc : dymoe_assign_precision(ctx, phase, importance, load, E, n_tiers, tier_count, tier_bits, floor_bits,
                                                            bits, rank, stream);
    }
    // (an assignment by whichever workgroup of the importance kernel ends last costs more than the launch it saves: the
    // device-wide fence each of them then needs took 20 us at 1357 tokens)
    dymoe_launch(ctx, DYMOE_K_TOKEN_NORM, dymoe::norm_and_zero_kernel, dim3((unsigned)((T + 3) / 4)), dim3(256), 0, st, xb, T, H,
                 token_score, (int32_t*)importance, load, E);
    DYMOE_HIP_LAUNCH_CHECK();
    dymoe_launch(ctx, DYMOE_K_IMPORTANCE, dymoe::importance_prefill_kernel,
                 dim3((unsigned)((T + dymoe::kImpTokens - 1) / dymoe::kImpTokens)), dim3(dymoe::kImpThreads), 0, st, idx, token_score, T,
                 E, k, k_hh, (int32_t*)importance, load);
    DYMOE_HIP_LAUNCH_CHECK();
    return dymoe_assign_precision(ctx, phase, importance, load, E, n_tiers, tier_count, tier_bits, floor_bits, bits, rank, stream);
}

int dymoe_assign_precision(dymoe_ctx* ctx, int phase, const void* importance,
                           const int32_t* load, int E, int n_tiers,
                           const int32_t* tier_count, const uint8_t* tier_bits, int floor_bits,
                           uint8_t* bits, int32_t* rank, void* stream)
{
    DYMOE_REQUIRE(importance && tier_count && tier_bits && bits);
    DYMOE_REQUIRE(phase == DYMOE_PHASE_PREFILL || phase == DYMOE_PHASE_DECODE);
    DYMOE_REQUIRE(E > 0 && n_tiers >= 1 && n_tiers <= DYMOE_MAX_TIERS);
    DYMOE_REQUIRE(floor_bits == 0 || floor_bits == 2 || floor_bits == 4 || floor_bits == 8 || floor_bits == 16);
    dymoe::TierTable tt;
    DYMOE_REQUIRE(dymoe::make_tier_table(E, n_tiers, tier_count, tier_bits, tt) == DYMOE_OK);
    if (E > DYMOE_MAX_EXPERTS) return DYMOE_ENOTSUP;
    if (!ctx) return DYMOE_ENOCTX;
    hipStream_t st = (hipStream_t)stream;
    // enough threads for eight lanes per expert, at most the 1024 of a workgroup
    unsigned threads = (unsigned)(((E * 8 + 63) / 64) * 64);
    if (threads > DYMOE_MAX_EXPERTS) threads = DYMOE_MAX_EXPERTS;
    if (phase == DYMOE_PHASE_PREFILL)
        dymoe_launch(ctx, DYMOE_K_ASSIGN, (dymoe::assign_precision_kernel<int32_t>), dim3(1), dim3(threads), 0, st,
                           (const int32_t*)importance, load, E, tt, floor_bits, bits, rank);
    else
        dymoe_launch(ctx, DYMOE_K_ASSIGN, (dymoe::assign_precision_kernel<float>), dim3(1), dim3(threads), 0, st,
                           (const float*)importance, load, E, tt, floor_bits, bits, rank);
    DYMOE_HIP_LAUNCH_CHECK();
    return DYMOE_OK;
}

}  // extern "C"
