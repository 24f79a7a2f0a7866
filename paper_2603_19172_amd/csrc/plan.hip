// Launches that prepare the grouped GEMM: the plan (counting sort of the (token, slot) pairs by expert, tile list, fp16
// copies of the activations), alone or with the experts' ranking and bit widths in front of it.
#include <math.h>

#include <type_traits>

#include "common.hpp"
#include "assign.hpp"
#include "plan_device.hpp"

namespace dymoe {

// One workgroup of 16 wavefronts.  Counting goes through one histogram per wavefront when they fit in LDS (E <=
// kPlanPrivE), so that the atomics of a popular expert do not queue up across the whole workgroup.  The counter's value
// before a pair was added is the pair's turn inside its wavefront: its position is (expert offset) + (pairs of the expert
// in earlier wavefronts) + turn, with no second pass of atomics.
// The workgroups behind the first one make the fp16 copies of x (prep_x) meanwhile: neither needs the other, and as a
// launch of their own the copies took 3 us (61 tokens of 2048) to 12 us (1357 of 4096) after the plan's 9 to 25.
__global__ __launch_bounds__(kPlanThreads) void plan_kernel(const int32_t* __restrict__ idx,
                                                            const uint8_t* __restrict__ bits,
                                                            const dymoe_expert_fmt* __restrict__ table, int P, int E,
                                                            int tile_m, int max_tiles, SplitRule splits,
                                                            int32_t* __restrict__ plan, unsigned* __restrict__ flags,
                                                            const uint16_t* __restrict__ x, long n16,
                                                            uint16_t* __restrict__ xh4, uint16_t* __restrict__ xh2,
                                                            uint16_t* __restrict__ xh8)
{
    if (blockIdx.x > 0) {
        const long i = (long)(blockIdx.x - 1) * kPlanThreads + threadIdx.x;
        if (i < n16) prep_x(x, i, xh4, xh2, xh8);
        return;
    }
    __shared__ int32_t s_count[DYMOE_MAX_EXPERTS];
    __shared__ int32_t s_off[DYMOE_MAX_EXPERTS + 1];
    __shared__ int32_t s_tile0[DYMOE_MAX_EXPERTS + 1];       // first tile of each expert
    __shared__ int32_t s_priv[kPlanWaves * kPlanPrivE];
    __shared__ __attribute__((aligned(16))) int32_t s_cnt[kPlanOrders * kPlanWaves];
    __shared__ uint8_t s_bits[DYMOE_MAX_EXPERTS];
    const PlanPtrs pp = plan_ptrs(plan, E, P);
    const int tid = threadIdx.x, wave = tid / kWave;
    const bool priv = E <= kPlanPrivE;
    // (the expert indices of a batch of pairs are requested together and looked at afterwards: one pair at a time, every
    // iteration waited a memory latency for its own index, 16 latencies per pass on the 128-expert layer)
    constexpr int kPlanBatch = 16;
    // up to 16 x 1024 pairs: a thread's indices and turns stay in registers from the counting pass to the scattering
    // pass, and are requested before the chain bits -> table entry -> its pointers; beyond, the scattering pass counts again
    const bool one_pass = P <= kPlanBatch * kPlanThreads;
    int es[kPlanBatch], turn[kPlanBatch];
    auto fetch = [&](int p0) {
#pragma unroll
        for (int u = 0; u < kPlanBatch; u++) {
            const int p = p0 + u * kPlanThreads;
            const int e = idx[min(p, P - 1)];
            es[u] = (p < P && e >= 0 && e < E) ? e : -1;
        }
    };
    if (one_pass) fetch(tid);
    for (int e = tid; e < E; e += kPlanThreads) {
        s_count[e] = 0;
        int b = bits[e];
        if (b == 16 || b == 8 || b == 4 || b == 2) {
            // a format the table does not hold: the expert is left out, as at 0 bits.  Whether it had pairs is not
            // known yet, but the decode path reports the same condition only for routed experts: checked below.
            if (!(dymoe_formats_held(table[e]) & b)) b = 0x80 | b;
        } else {
            b = 0;
        }
        s_bits[e] = (uint8_t)b;
    }
    if (priv)
        for (int i = tid; i < kPlanWaves * E; i += kPlanThreads) s_priv[i] = 0;
    __syncthreads();
    for (int p0 = tid; p0 < P || p0 == tid; p0 += kPlanBatch * kPlanThreads) {
        if (!one_pass) fetch(p0);
#pragma unroll
        for (int u = 0; u < kPlanBatch; u++)
            if (es[u] >= 0) turn[u] = atomicAdd(priv ? &s_priv[wave * E + es[u]] : &s_count[es[u]], 1);
    }
    __syncthreads();
    for (int e = tid; e < E; e += kPlanThreads) {
        const int total = priv ? plan_gather(e, E, s_priv) : s_count[e];
        const int b = s_bits[e];
        if ((b & 0x80) && total > 0) atomicOr(flags, DYMOE_FLAG_FORMAT_MISSING);   // routed to, selected format absent: say so
        s_count[e] = (b != 0 && !(b & 0x80)) ? total : 0;                           // ... and leave its pairs out
    }
    __syncthreads();
    plan_scan(E, tile_m, s_count, s_bits, s_off, s_tile0, splits, pp);
    if (s_tile0[E] <= kPlanShortList) plan_tile_list(E, tile_m, s_count, s_bits, s_off, s_tile0, s_cnt, pp);
    else plan_tile_list_long(E, tile_m, s_count, s_bits, s_off, s_tile0, pp.tiles + 4 * (size_t)max_tiles, pp);
    plan_tables(E, s_count, s_bits, s_off, pp);
    __syncthreads();
    if (!priv && !one_pass) {
        for (int e = tid; e < E; e += kPlanThreads) s_count[e] = 0;    // reused as the scatter cursor
        __syncthreads();
    }
    // order inside an expert is arbitrary: every row of a tile is computed independently
    for (int p0 = tid; p0 < P || p0 == tid; p0 += kPlanBatch * kPlanThreads) {
        if (!one_pass) fetch(p0);
#pragma unroll
        for (int u = 0; u < kPlanBatch; u++) {
            const int e = es[u];
            if (e < 0 || s_bits[e] == 0 || (s_bits[e] & 0x80)) continue;
            int pos = s_off[e];
            if (one_pass) pos += turn[u] + (priv ? s_priv[wave * E + e] : 0);
            else pos += atomicAdd(priv ? &s_priv[wave * E + e] : &s_count[e], 1);
            pp.perm[pos] = p0 + u * kPlanThreads;
        }
    }
}

int plan_launch(dymoe_ctx* ctx, const void* x, const int32_t* idx, const uint8_t* bits, const dymoe_expert_fmt* table, int T, int H,
                int E, int k, const SplitRule& splits, const FfnLayout& L, char* ws, hipStream_t st)
{
    uint16_t* xh4 = reinterpret_cast<uint16_t*>(ws + L.xh);
    uint16_t* xh2 = xh4 + round256((size_t)T * H * 2) / 2;
    uint16_t* xh8 = xh2 + round256((size_t)T * H * 2) / 2;
    const long n16 = (long)T * H / 16;
    dymoe_launch(ctx, DYMOE_K_PLAN, plan_kernel, dim3((unsigned)(1 + (n16 + kPlanThreads - 1) / kPlanThreads)), dim3(kPlanThreads), 0,
                 st, idx, bits, table, T * k, E, ffn_tile_rows(T, E, k), L.max_tiles, splits, reinterpret_cast<int32_t*>(ws + L.plan), ctx->device_flags,
                 (const uint16_t*)x, n16, xh4, xh2, xh8);
    DYMOE_HIP_LAUNCH_CHECK();
    return DYMOE_OK;
}

// Ranking, bit widths and plan in one launch, for a layer's own step: dymoe_rank_experts' results (importance, load, bits,
// rank; the norms come from the router's launch) and the plan of those bits, by the first workgroup; the others make the
// fp16 copies of x that the tiers' formats can ask for.  The pairs are counted once, for the load and for the plan.
// Bound: latency, a chain of about a dozen hand-overs through LDS behind two trips to memory.  us among the other
// launches of a step, and the launches it stands for (norms, importance, assignment, plan): 16 tokens x 2 of 8 experts 6.5 for
// 3.7 + 5.5, 61 x 8 of 128 (decode) 9.5 for 5.8 + 9.8, 512 x 2 of 8 11 for 5.6 + 5.5 + 4.9 + 14, 2048 x 8 of 128 21 for
// 5.1 + 9.7 + 6.1 + 31.  (There, 4 to 5 of the 21 are the first loads, behind the copies' traffic.)
//   prefill  up to 256 tokens rank themselves by counting, as in importance_block_kernel; beyond, the k_hh-th largest score
//            is found by a radix selection (11 bits at a time) and the heavy tokens are those above it, ties in token order
//   decode   mean probability in token order, as in importance_block_kernel
struct RankPlanArgs {
    const int32_t* idx;
    const float* score;                // prefill
    const float* probs;                // decode
    int T, E, k, k_hh, P;
    uint32_t div_k;                    // ceil(2^32 / k): p / k of a pair p < 2^16
    void* importance;
    int32_t* load;
    TierTable tiers;
    int floor_bits;
    uint8_t* bits;
    int32_t* rank;
    const dymoe_expert_fmt* table;
    int formats;                       // sum of the bit widths the tiers can assign
    int tile_m;
    SplitRule splits;
    int32_t* plan;
    unsigned* flags;
    const uint16_t* x;
    long n16;
    uint16_t *xh4, *xh2, *xh8;
};

constexpr int kRpMaxE = kPlanPrivE;
constexpr int kRpMaxPairs = 32 * kPlanThreads;
static_assert(kRpMaxE <= 256 && kRpMaxPairs <= 1 << 16, "an expert in 8 bits, a pair in 16");
constexpr int kRpMaxTokens = 8192;
constexpr int kRpDirect = 256;         // prefill tokens that rank themselves by counting
constexpr int kRpBuf = 8192;           // scores, staged probabilities, then the grouped pairs (16 bits each) and the tile list
constexpr int kRpDigit = 11;           // bits of the radix selection's digits

// Which of the T > kRpDirect tokens are heavy (fewer than k_hh precede them: larger score, or the same and a smaller
// index): s_key, the scores' bits + 1 (0 for NaN, which nothing precedes and which precedes nothing), become flags.
// s_hist: zeros, s_sel[0]: -1.
__device__ __forceinline__ void mark_heavy(uint32_t* s_key, int T, int k_hh, int32_t* s_hist, int32_t* s_wave, int32_t* s_sel)
{
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    uint32_t prefix = 0;               // the digits of the k_hh-th largest key found so far
    int need = k_hh, shift = 32, ties = 0;
    bool all = false;
    while (shift > 0) {
        const int bits = shift == 10 ? 10 : kRpDigit, below = shift - bits;
        for (int t = tid; t < T; t += kPlanThreads) {
            const uint32_t key = s_key[t];
            if (key != 0 && (shift == 32 || (key >> shift) == prefix)) {
                // (nearly all scores share their first digit: those equal to the first lane's are added by one lane)
                const int d = (int)((key >> below) & ((1u << bits) - 1));
                const int d0 = __builtin_amdgcn_readfirstlane(d);
                const unsigned long long same = __ballot(d == d0);
                if (d != d0) atomicAdd(&s_hist[d], 1);
                else if (lane == __ffsll((long long)same) - 1) atomicAdd(&s_hist[d0], __popcll(same));
            }
        }
        __syncthreads();
        // keys above each digit, two digits a thread; the counters are zeros again for the next round
        const int c0 = s_hist[2 * tid], c1 = s_hist[2 * tid + 1];
        s_hist[2 * tid] = s_hist[2 * tid + 1] = 0;
        const int incl = wave_scan_dpp_i32(c0 + c1);
        if (lane == kWave - 1) s_wave[wave] = incl;
        __syncthreads();
        int above = c0 + c1 - incl;    // all of this and the later wavefronts' keys less those up to this thread's
#pragma unroll
        for (int wv = 0; wv < kPlanWaves; wv++) above += (wv >= wave) ? s_wave[wv] : 0;
        above -= c0 + c1;
        if (above < need && need <= above + c1) {
            s_sel[0] = 2 * tid + 1;
            s_sel[1] = above;
            s_sel[2] = c1;
        } else if (above + c1 < need && need <= above + c1 + c0) {
            s_sel[0] = 2 * tid;
            s_sel[1] = above + c1;
            s_sel[2] = c0;
        }
        __syncthreads();
        const int digit = s_sel[0];
        if (digit < 0) {               // (first digit only) no more keys than heavy tokens asked for
            all = true;
            break;
        }
        need -= s_sel[1];
        prefix = (prefix << bits) | (uint32_t)digit;
        shift = below;
        ties = s_sel[2];
        if (ties == need) break;       // every key with these digits is heavy
    }
    if (all || ties == need) {
        for (int t = tid; t < T; t += kPlanThreads) {
            const uint32_t key = s_key[t];
            s_key[t] = (all || key == 0 || (key >> shift) >= prefix) ? 1u : 0u;
        }
        return;
    }
    // more tokens of exactly the k_hh-th largest score than are heavy: the first `need` of them
    const int trips = (T + kPlanThreads - 1) / kPlanThreads;
    for (int u = 0; u < trips; u++) {
        const int t = tid + u * kPlanThreads;
        const unsigned long long eq = __ballot(t < T && s_key[min(t, T - 1)] == prefix);
        if (lane == 0) s_hist[u * kPlanWaves + wave] = __popcll(eq);
    }
    __syncthreads();
    for (int u = 0; u < trips; u++) {
        const int t = tid + u * kPlanThreads;
        const uint32_t key = s_key[min(t, T - 1)];
        const unsigned long long eq = __ballot(t < T && key == prefix);
        int before = __popcll(eq & ((1ull << lane) - 1));
        for (int i = 0; i < u * kPlanWaves + wave; i++) before += s_hist[i];
        if (t < T) s_key[t] = (key == 0 || key > prefix || (key == prefix && before < need)) ? 1u : 0u;
    }
}

// NP: pairs per thread, kept in registers.
template <bool PREFILL, int NP>
__global__ __launch_bounds__(kPlanThreads) void rank_plan_kernel(const RankPlanArgs a)
{
    if (blockIdx.x > 0) {
        const long i = (long)(blockIdx.x - 1) * kPlanThreads + threadIdx.x;
        if (i < a.n16) prep_x(a.x, i, a.xh4, a.xh2, a.xh8);
        return;
    }
    using ImpT = typename std::conditional<PREFILL, int32_t, float>::type;
    __shared__ int32_t s_count[kRpMaxE], s_load[kRpMaxE], s_off[kRpMaxE + 1], s_tile0[kRpMaxE + 1];
    __shared__ ImpT s_imp[kRpMaxE];
    __shared__ int32_t s_priv[kPlanWaves * kRpMaxE];
    __shared__ __attribute__((aligned(16))) uint32_t s_buf[kRpBuf];
    __shared__ int32_t s_hist[PREFILL ? 1 << kRpDigit : 1], s_wave[kPlanWaves], s_sel[4], s_none[kWave];
    __shared__ __attribute__((aligned(16))) int32_t s_cnt[kPlanOrders * kPlanWaves];
    static_assert(2 * kPlanThreads == (1 << kRpDigit), "two digits a thread");
    __shared__ __attribute__((aligned(16))) uint64_t s_key[kRpMaxE];
    __shared__ int32_t s_nan;
    __shared__ uint8_t s_bits[kRpMaxE];
    const int T = a.T, E = a.E, k = a.k, P = a.P;
    const PlanPtrs pp = plan_ptrs(a.plan, E, P);
    const int tid = threadIdx.x, wave = tid / kWave;
    // everything memory holds is requested first
    int es[NP];                                                // expert (-1: none), from 8 bits on the pair's turn
#pragma unroll
    for (int u = 0; u < NP; u++) {
        const int p = tid + u * kPlanThreads;
        const int e = a.idx[min(p, P - 1)];
        es[u] = (p < P && e >= 0 && e < E) ? e : -1;
    }
    constexpr int kStage = kRpBuf / kPlanThreads;
    const int stage_tokens = kRpBuf / E;                       // decode: tokens whose probabilities s_buf takes
    float staged[PREFILL ? 1 : kStage];
    if constexpr (PREFILL) {
        for (int t = tid; t < max(T, kRpDirect); t += kPlanThreads) {
            const float s = (t < T) ? a.score[t] : -INFINITY;  // (up to kRpDirect: past every token, never counted)
            s_buf[t] = (T <= kRpDirect) ? __float_as_uint(s) : (s == s ? __float_as_uint(s) + 1u : 0u);
        }
    } else {
        const int n = min(stage_tokens, T) * E;
#pragma unroll
        for (int u = 0; u < kStage; u++) staged[u] = a.probs[min(u * kPlanThreads + tid, n - 1)];
    }
    int have = 0;                                              // formats of expert tid that the table holds
    if (tid < E) {
        have = dymoe_formats_held(a.table[tid]);
        s_imp[tid] = 0;
    }
    for (int i = tid; i < kPlanWaves * E; i += kPlanThreads) s_priv[i] = 0;
    if (tid == 0) s_nan = 0;
    if constexpr (PREFILL) {
        s_hist[2 * tid] = s_hist[2 * tid + 1] = 0;
        if (tid == 0) s_sel[0] = -1;
    }
    __syncthreads();
    {
        // (no branches, so that all are under way together: a lane without a pair counts in a place of its own)
        int turn[NP];
#pragma unroll
        for (int u = 0; u < NP; u++) turn[u] = atomicAdd(es[u] >= 0 ? &s_priv[wave * E + es[u]] : &s_none[tid & (kWave - 1)], 1);
#pragma unroll
        for (int u = 0; u < NP; u++) es[u] = es[u] >= 0 ? es[u] | (turn[u] << 8) : -1;
    }
    if constexpr (PREFILL) {
        if (a.k_hh <= 0) {
            __syncthreads();
            for (int t = tid; t < T; t += kPlanThreads) s_buf[t] = 0u;
        } else if (T <= kRpDirect) {
            const float* s_score = reinterpret_cast<const float*>(s_buf);
            int lanes = 64;
            while (lanes * T > kPlanThreads) lanes >>= 1;
            const int t = tid / lanes, part = tid % lanes;
            int before = 0;
            if (t < T) {
                const float mine = s_score[t];
                for (int j = 4 * part; j < T; j += 4 * lanes) {
                    const float4 s4 = *reinterpret_cast<const float4*>(s_score + j);
                    before += (s4.x > mine || (s4.x == mine && j + 0 < t)) ? 1 : 0;
                    before += (s4.y > mine || (s4.y == mine && j + 1 < t)) ? 1 : 0;
                    before += (s4.z > mine || (s4.z == mine && j + 2 < t)) ? 1 : 0;
                    before += (s4.w > mine || (s4.w == mine && j + 3 < t)) ? 1 : 0;
                }
            }
            for (int o = 1; o < lanes; o <<= 1) before += __shfl_xor(before, o, kWave);
            __syncthreads();                                   // the scores have been read: their place takes the flags
            if (t < T && part == 0) s_buf[t] = before < a.k_hh ? 1u : 0u;
        } else {
            mark_heavy(s_buf, T, a.k_hh, s_hist, s_wave, s_sel);
        }
    } else {
        float* const s_prob = reinterpret_cast<float*>(s_buf);
        float g = 0.0f;                                        // of expert tid
        for (int t0 = 0; t0 < T; t0 += stage_tokens) {
            const int n = min(stage_tokens, T - t0);
            if (t0 > 0) {
#pragma unroll
                for (int u = 0; u < kStage; u++) staged[u] = a.probs[(size_t)t0 * E + min(u * kPlanThreads + tid, n * E - 1)];
                __syncthreads();                               // the previous trip's have been read
            }
#pragma unroll
            for (int u = 0; u < kStage; u++) s_prob[u * kPlanThreads + tid] = staged[u];
            __syncthreads();
            if (tid < E)
#pragma unroll 8
                for (int t = 0; t < n; t++) g += s_prob[t * E + tid];
        }
        if (tid < E) s_imp[tid] = (T <= 1) ? g : g / (float)T;
    }
    __syncthreads();
    if (tid < E) s_load[tid] = plan_gather(tid, E, s_priv);
    if constexpr (PREFILL) {
        uint32_t heavy[NP];
#pragma unroll
        for (int u = 0; u < NP; u++) {
            const uint32_t p = (uint32_t)(tid + u * kPlanThreads);
            const uint32_t t = (k == 1) ? p : __umulhi(p, a.div_k);
            heavy[u] = s_buf[min(t, (uint32_t)T - 1)];
        }
#pragma unroll
        for (int u = 0; u < NP; u++)
            if (es[u] >= 0 && heavy[u]) atomicAdd(&s_imp[es[u] & 255], 1);
    }
    __syncthreads();
    if (tid < E) {
        a.load[tid] = s_load[tid];
        reinterpret_cast<ImpT*>(a.importance)[tid] = s_imp[tid];
    }
    bool whole = true;                                         // no NaN among the importances
    if constexpr (!PREFILL) {
        if (tid < E && !(s_imp[tid] == s_imp[tid])) s_nan = 1;
        __syncthreads();
        whole = s_nan == 0;
    }
    if (whole) {
        // importance, load and index of an expert as one number: expert e's position is the count of larger ones.  8 lanes
        // (4 from 129 experts on) share an expert, two rivals a read.
        if (tid < kRpMaxE) {
            uint32_t hi = 0;
            if (tid < E) {
                if constexpr (PREFILL) hi = (uint32_t)s_imp[tid];
                else hi = __float_as_uint(s_imp[tid]);         // (not negative: the order of the bits)
            }
            s_key[tid] = tid < E ? ((uint64_t)hi << 32) | ((uint32_t)s_load[tid] << 8) | (uint32_t)(255 - tid) : 0;
        }
        __syncthreads();
        const int lg = E <= kPlanThreads / 8 ? 3 : 2, e = tid >> lg;
        const uint64_t mine = s_key[min(e, kRpMaxE - 1)];
        int pos = 0;
#pragma unroll 2
        for (int j = 2 * (tid & ((1 << lg) - 1)); j < E; j += 2 << lg) {
            const ulonglong2 r = *reinterpret_cast<const ulonglong2*>(s_key + j);
            pos += (r.x > mine ? 1 : 0) + (r.y > mine ? 1 : 0);
        }
        pos += __builtin_amdgcn_update_dpp(0, pos, 0xB1, 0xF, 0xF, true);       // the quad's lanes, then the other quad's
        pos += __builtin_amdgcn_update_dpp(0, pos, 0x4E, 0xF, 0xF, true);
        if (lg == 3) pos += __builtin_amdgcn_update_dpp(0, pos, 0x141, 0xF, 0xF, true);
        if (e < E && (tid & ((1 << lg) - 1)) == 0) {
            s_bits[e] = (uint8_t)tier_bits_at(pos, a.tiers, a.floor_bits);
            a.rank[e] = pos;
        }
    } else {
        assign_all<ImpT>(kPlanThreads, E, s_imp, s_load, a.tiers, a.floor_bits, s_bits, a.rank);
    }
    __syncthreads();
    if (tid < E) {
        const int total = s_load[tid];
        int b = s_bits[tid];
        a.bits[tid] = (uint8_t)b;
        if (b != 0 && !(have & b)) {                           // the table lacks the format: left out, as at 0 bits
            if (total > 0) atomicOr(a.flags, DYMOE_FLAG_FORMAT_MISSING);
            b = 0;
        }
        s_bits[tid] = (uint8_t)b;
        s_count[tid] = b ? total : 0;
    }
    __syncthreads();
    plan_scan(E, a.tile_m, s_count, s_bits, s_off, s_tile0, a.splits, pp);
    // the wavefronts' first positions among all pairs; negative where the expert is left out
    for (int i = tid; i < kPlanWaves * E; i += kPlanThreads) {
        const int e = i % E;
        s_priv[i] = s_bits[e] ? s_priv[i] + s_off[e] : -1;
    }
    __syncthreads();
    // grouped in LDS and written out whole: a store of 64 pairs straight to their places would touch as many cache lines
    uint16_t* const s_perm = reinterpret_cast<uint16_t*>(s_buf);
    constexpr bool kInLds = NP * kPlanThreads <= 2 * kRpBuf;
    int first[NP];
#pragma unroll
    for (int u = 0; u < NP; u++) first[u] = s_priv[wave * E + min(es[u] & 255, E - 1)];
#pragma unroll
    for (int u = 0; u < NP; u++) {
        if (es[u] < 0 || first[u] < 0) continue;
        const int pos = first[u] + (es[u] >> 8);
        if constexpr (kInLds) s_perm[pos] = (uint16_t)(tid + u * kPlanThreads);
        else pp.perm[pos] = tid + u * kPlanThreads;
    }
    __syncthreads();
    if constexpr (kInLds) {
        const int n = s_off[E];
#pragma unroll
        for (int u = 0; u < NP; u++) {
            const int i = tid + u * kPlanThreads;
            if (i < n) pp.perm[i] = s_perm[i];
        }
    }
    plan_tables(E, s_count, s_bits, s_off, pp);
    plan_tile_list(E, a.tile_m, s_count, s_bits, s_off, s_tile0, s_cnt, pp);
}

bool rank_plan_fits(int T, int E, int k)
{
    return E <= kRpMaxE && T <= kRpMaxTokens && (long)T * k <= kRpMaxPairs && k <= 256;
}

int rank_plan_launch(dymoe_ctx* ctx, bool prefill, const void* x, const int32_t* idx, const float* probs, const float* score, int T, int H,
                     int E, int k, int k_hh, const TierTable& tiers, int floor_bits, const dymoe_expert_fmt* table, void* importance,
                     int32_t* load, uint8_t* bits, int32_t* rank, const SplitRule& splits, const FfnLayout& L, char* ws, hipStream_t st)
{
    RankPlanArgs a = {};
    a.idx = idx; a.score = score; a.probs = probs;
    a.T = T; a.E = E; a.k = k; a.k_hh = k_hh; a.P = T * k;
    a.div_k = (uint32_t)((((uint64_t)1 << 32) + (uint64_t)k - 1) / (uint64_t)k);
    a.importance = importance; a.load = load; a.tiers = tiers; a.floor_bits = floor_bits; a.bits = bits; a.rank = rank;
    a.table = table;
    for (int i = 0; i < tiers.n; i++)
        if (tiers.count[i] > 0) a.formats |= tiers.bits[i] < floor_bits ? floor_bits : tiers.bits[i];
    a.tile_m = ffn_tile_rows(T, E, k);
    a.splits = splits;
    a.plan = reinterpret_cast<int32_t*>(ws + L.plan);
    a.flags = ctx->device_flags;
    a.x = (const uint16_t*)x;
    a.n16 = (long)T * H / 16;
    uint16_t* const xh4 = reinterpret_cast<uint16_t*>(ws + L.xh);
    uint16_t* const xh2 = xh4 + round256((size_t)T * H * 2) / 2;
    uint16_t* const xh8 = xh2 + round256((size_t)T * H * 2) / 2;
    a.xh4 = (a.formats & 4) ? xh4 : nullptr;
    a.xh2 = (a.formats & 2) ? xh2 : nullptr;
    a.xh8 = (a.formats & 8) ? xh8 : nullptr;
    const long copies = (a.formats & 14) ? (a.n16 + kPlanThreads - 1) / kPlanThreads : 0;
    auto go = [&](auto kernel) {
        dymoe_launch(ctx, DYMOE_K_PLAN, kernel, dim3((unsigned)(1 + copies)), dim3(kPlanThreads), 0, st, a);
    };
    if (a.P <= kPlanThreads) prefill ? go(rank_plan_kernel<true, 1>) : go(rank_plan_kernel<false, 1>);
    else if (a.P <= 4 * kPlanThreads) prefill ? go(rank_plan_kernel<true, 4>) : go(rank_plan_kernel<false, 4>);
    else if (a.P <= 16 * kPlanThreads) prefill ? go(rank_plan_kernel<true, 16>) : go(rank_plan_kernel<false, 16>);
    else prefill ? go(rank_plan_kernel<true, 32>) : go(rank_plan_kernel<false, 32>);
    DYMOE_HIP_LAUNCH_CHECK();
    return DYMOE_OK;
}

}  // namespace dymoe
