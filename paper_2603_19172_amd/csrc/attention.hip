// Attention-derived token score (paper Sec. 4.2.1, first equation):
//   s_i = (1/Hh) sum_h a_i^(h),   a_i^(h) = (1/T) sum_q P^(h)[q, i],
// the attention token i receives, averaged over queries and heads, where
// P^(h) = softmax over keys of (q_q . k_i) * scale, keys after the query masked
// out when `causal`.  The probabilities are never stored: one pass over the keys
// gives every query's softmax maximum and normaliser, a second pass rebuilds the
// logits tile by tile and adds exp(logit - max) / normaliser into per-key sums.
//
// Both passes compute tiles of S^T = K Q^T (keys down, queries across) with
// v_mfma_f32_32x32x16_bf16.  Queries and keys are [token][head][d] rows, so a
// lane's 16-byte pieces of a row are at once the A operand (keys) and the B
// operand (queries): for short sequences nothing goes through LDS (long ones
// share the streamed operand between wavefronts, see below).  In the result a lane holds one
// query (column) and 16 keys (rows): the softmax statistics of a query and the
// running per-key sums both stay inside a lane until the very end.
#include <type_traits>

#include "attention_rule.hpp"
#include "common.hpp"

namespace dymoe {

constexpr int kAtThreads = kAtWaves * kWave;

// One lane's share of a 32-token fragment of one head (D columns): lane (ln, kb)
// holds row ln; piece c covers columns 32 (c / 2) + 16 kb + 8 (c % 2) .. + 7, i.e.
// 32 contiguous bytes per pair of pieces.  Queries and keys use the same
// column order, so the contraction is over matching columns.
template <int D>
struct AtFrag {
    uint4 c[D / 16];
};

template <int D>
__device__ __forceinline__ void load_frag(const uint16_t* __restrict__ head_base, long row_stride, int row,
                                          int kb, AtFrag<D>& f)
{
    const uint16_t* p = head_base + (long)row * row_stride + kb * 16;
#pragma unroll
    for (int c2 = 0; c2 < D / 32; c2++) {
        f.c[2 * c2] = load_global<uint4>(p + c2 * 32);
        f.c[2 * c2 + 1] = load_global<uint4>(p + c2 * 32 + 8);
    }
}

// S^T tile: rows = the 32 keys of fk, columns = the 32 queries of fq.
// Lane (ln, kb), register i: key 8 (i / 4) + 4 kb + i % 4, query ln.
template <int D>
__device__ __forceinline__ float16_t logits_tile(const AtFrag<D>& fk, const AtFrag<D>& fq)
{
    float16_t acc;
#pragma unroll
    for (int i = 0; i < 16; i++) acc[i] = 0.0f;
#pragma unroll
    for (int c = 0; c < D / 16; c++)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, fk.c[c]),
                                                      __builtin_bit_cast(bf16x8_t, fq.c[c]), acc, 0, 0, 0);
    return acc;
}

__device__ __forceinline__ int tile_key(int kf, int kb, int i) { return kf * 32 + 8 * (i >> 2) + 4 * kb + (i & 3); }

// Workgroup -> (fragment, head).  Workgroups are handed to the 8 XCDs in turn
// (linear id modulo 8), each with an L2 of its own: when the heads divide
// evenly, every XCD gets whole heads, so that one head's queries and keys are
// read through one L2 instead of all eight.
__device__ __forceinline__ void fragment_and_head(int nfrag, int n_heads, int& frag, int& head)
{
    const int lin = blockIdx.x + gridDim.x * blockIdx.y;      // grid = (nfrag, n_heads)
    if (n_heads % 8 == 0) {
        const int xcd = lin & 7, j = lin >> 3, per = n_heads >> 3;
        head = xcd * per + j / nfrag;
        frag = j - (j / nfrag) * nfrag;
    } else {
        frag = blockIdx.x;
        head = blockIdx.y;
    }
}

constexpr float kMasked = -1.0e30f;     // finite stand-in for minus infinity: no NaN from (-inf) - (-inf)

// Pass 1.  A workgroup owns 32 queries of one head; its four wavefronts take
// every fourth key fragment each (interleaved, so a causal mask leaves them
// equal shares) and keep a running maximum m and sum l of exp2(logit' - m),
// logit' = logit * scale * log2(e); the four (m, l) pairs of a query are merged
// through LDS in wavefront order.  stats[h][q] = (m, 1 / l).
template <int D>
__global__ __launch_bounds__(kAtThreads) void attn_rowstats_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, int T, int n_heads, int group,
    float scale_log2, int causal, float2* __restrict__ stats)
{
    __shared__ float2 s_ml[kAtWaves][32];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int ln = lane & 31, kb = lane >> 5;
    const int nfrag = (T + 31) >> 5;
    int qf, h;
    fragment_and_head(nfrag, n_heads, qf, h);
    const long q_stride = (long)n_heads * D, k_stride = (long)(n_heads / group) * D;
    const uint16_t* qh = q + (long)h * D;
    const uint16_t* kh = k + (long)(h / group) * D;
    const int query = qf * 32 + ln;
    AtFrag<D> fq, fk, fn;
    load_frag<D>(qh, q_stride, min(query, T - 1), kb, fq);     // rows past the end re-read the last token; masked below
    const int kf_last = causal ? qf : nfrag - 1;
    load_frag<D>(kh, k_stride, min(wave * 32 + ln, T - 1), kb, fk);
    float m = kMasked, l = 0.0f;
    for (int kf = wave; kf <= kf_last; kf += kAtWaves) {
        const int kn = (kf + kAtWaves <= kf_last) ? kf + kAtWaves : kf;   // the next fragment is requested before this one is used
        load_frag<D>(kh, k_stride, min(kn * 32 + ln, T - 1), kb, fn);
        const float16_t acc = logits_tile<D>(fk, fq);
        float sv[16];
        float mx = m;
#pragma unroll
        for (int i = 0; i < 16; i++) {
            const int key = tile_key(kf, kb, i);
            const bool ok = key < T && (!causal || key <= query);
            sv[i] = ok ? acc[i] * scale_log2 : kMasked;
            mx = fmaxf(mx, sv[i]);
        }
        float add = 0.0f;
#pragma unroll
        for (int i = 0; i < 16; i++) add += (sv[i] > 0.5f * kMasked) ? __builtin_amdgcn_exp2f(sv[i] - mx) : 0.0f;
        l = l * __builtin_amdgcn_exp2f(m - mx) + add;
        m = mx;
        fk = fn;
    }
    // the two halves of the keys (kb = 0, 1) of this query
    const float m2 = __shfl_xor(m, 32, kWave), l2 = __shfl_xor(l, 32, kWave);
    float M = fmaxf(m, m2);
    float L = l * __builtin_amdgcn_exp2f(m - M) + l2 * __builtin_amdgcn_exp2f(m2 - M);
    if (kb == 0) s_ml[wave][ln] = make_float2(M, L);
    __syncthreads();
    if (wave == 0 && kb == 0 && query < T) {
        M = s_ml[0][ln].x;
#pragma unroll
        for (int w = 1; w < kAtWaves; w++) M = fmaxf(M, s_ml[w][ln].x);
        L = 0.0f;
#pragma unroll
        for (int w = 0; w < kAtWaves; w++) L += s_ml[w][ln].y * __builtin_amdgcn_exp2f(s_ml[w][ln].x - M);
        stats[(long)h * T + query] = make_float2(M, 1.0f / L);
    }
}

// Pass 2.  A workgroup owns 32 keys of one head; its wavefronts take every fourth
// query fragment among those that see the keys:
// partial[h][key] = sum_q exp2(logit' - m_q) / l_q, the four wavefronts' sums added in order.
template <int D>
__global__ __launch_bounds__(kAtThreads) void attn_colsum_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, int T, int n_heads, int group,
    float scale_log2, int causal, const float2* __restrict__ stats, float* __restrict__ partial)
{
    __shared__ float s_col[kAtWaves][32];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int ln = lane & 31, kb = lane >> 5;
    const int nfrag = (T + 31) >> 5;
    int kf, h;
    fragment_and_head(nfrag, n_heads, kf, h);
    const long q_stride = (long)n_heads * D, k_stride = (long)(n_heads / group) * D;
    const uint16_t* qh = q + (long)h * D;
    const uint16_t* kh = k + (long)(h / group) * D;
    const float2* sh = stats + (long)h * T;
    AtFrag<D> fk, fq, fn;
    load_frag<D>(kh, k_stride, min(kf * 32 + ln, T - 1), kb, fk);
    const int qf_first = (causal ? kf : 0) + wave;
    load_frag<D>(qh, q_stride, min(qf_first * 32 + ln, T - 1), kb, fq);
    float2 st = sh[min(qf_first * 32 + ln, T - 1)];
    float col[16];
#pragma unroll
    for (int i = 0; i < 16; i++) col[i] = 0.0f;
    for (int qf = qf_first; qf < nfrag; qf += kAtWaves) {
        const int qn = (qf + kAtWaves < nfrag) ? qf + kAtWaves : qf;
        load_frag<D>(qh, q_stride, min(qn * 32 + ln, T - 1), kb, fn);
        const float2 stn = sh[min(qn * 32 + ln, T - 1)];
        const float16_t acc = logits_tile<D>(fk, fq);
        const int query = qf * 32 + ln;
#pragma unroll
        for (int i = 0; i < 16; i++) {
            const int key = tile_key(kf, kb, i);
            const bool ok = query < T && key < T && (!causal || key <= query);
            const float p = __builtin_amdgcn_exp2f(acc[i] * scale_log2 - st.x) * st.y;
            col[i] += ok ? p : 0.0f;
        }
        fq = fn;
        st = stn;
    }
    // sum over the 32 queries held by the lanes of each half
#pragma unroll
    for (int i = 0; i < 16; i++) {
        float v = col[i];
#pragma unroll
        for (int o = 16; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
        col[i] = v;
    }
    if (ln == 0) {
#pragma unroll
        for (int i = 0; i < 16; i++) s_col[wave][tile_key(0, kb, i)] = col[i];
    }
    __syncthreads();
    if (threadIdx.x < 32) {
        const int key = kf * 32 + threadIdx.x;
        float v = s_col[0][threadIdx.x];
#pragma unroll
        for (int w = 1; w < kAtWaves; w++) v += s_col[w][threadIdx.x];
        if (key < T) partial[(long)h * T + key] = v;
    }
}

// ----------------------------------------------------------------------------
// Long sequences: the streamed operand goes through LDS.  A workgroup of eight wavefronts (or four) owns OWNERS x 64 tokens: each
// wavefront keeps two 32-token fragments in registers, so that what it reads from LDS feeds two products (with one fragment
// the reads alone took the 128 bytes a cycle that LDS has), and the WAVES / OWNERS wavefronts that own the same tokens share
// the stream, two of a trip's fragments each; their statistics or sums meet in LDS at the end.
// 16-byte chunk c of row r lies at chunk position c ^ (r mod chunks-per-row), so that the operand reads of 16 consecutive
// rows fall on different banks.  The rows go from memory to LDS directly: through registers, the addresses and the stores took a
// quarter of the vector instructions.
// Bound: per 32 x 32 logits at d = 128 256 cycles of matrix instructions beside 32 multiply-adds and 16 exponentials (8 cycles each)
// a lane, 256 cycles as well, and the chip's power allows both together at 1.7 GHz only (a loop of nothing else takes 206 ns per
// 32 x 32, these kernels 230; the order of the instructions moves that by 2 %).  The whole score, 32 / 8 heads, d = 128, with one
// fragment per wavefront, four wavefronts in a block of 128 tokens and every fragment's maximum -> so: 4096 tokens causal 194 -> 160 us,
// unmasked 340 -> 276, 1024 causal 41 -> 28; 4096 x 6 heads 135 -> 77.
// At d = 64 the products are half of that and the vector work is the bound, whose latencies two wavefronts a SIMD leave open: where the
// blocks are many, three workgroups of four wavefronts share a compute unit (causal, one workgroup of eight / so: 2500 x 64 heads 123 -> 89 us,
// 4096 x 48 200 -> 153; with one fragment per wavefront 107 and 189).
// At d = 128 registers and LDS leave room for two such workgroups: no more wavefronts than in one of eight, but one that ends or waits at
// its barriers no longer idles the unit, and half as long a chain fills the chip more evenly (causal, one of eight / so: 1600 x 44 66.1 ->
// 53.6 us, unmasked 110 -> 92.2).
template <int D, int OWNERS, int WAVES>
struct AtWide {
    static constexpr int kStreams = WAVES / OWNERS;
    static constexpr int kEach = 2;                             // streamed fragments per wavefront and trip
    static constexpr int kFrags = kEach * kStreams;
    static constexpr int kRows = 32 * kFrags;
    static constexpr int kFragBytes = 32 * D * 2;
    static constexpr int kBufBytes = kRows * D * 2;
    static constexpr int kBufs = (3 * kBufBytes <= WAVES * 16 * 1024) ? 3 : 2;     // a trip's rows are requested kBufs - 1 trips ahead
    static constexpr int kUnitRows = 1024 / (D * 2);            // rows that one copy of a wavefront fills
    static constexpr int kUnits = kRows / kUnitRows / WAVES;        // copies per wavefront and trip
    const char* base;           // the head's first row
    uint32_t stride;            // bytes; a trip's 256 rows at most stay below 2^32 (65535 heads)
    uint32_t row, chunk;        // this lane's row of the wavefront's first unit and its bytes' place in the row
    uint32_t lds;               // LDS address of that unit, buffer 0

    __device__ __forceinline__ AtWide(const uint16_t* head, int n_heads, const char* s_buf, int wave, int lane)
    {
        constexpr int CH = D / 8;
        base = (const char*)head;
        stride = (uint32_t)n_heads * (D * 2);
        row = wave * kUnitRows + lane / CH;
        chunk = ((lane ^ row) & (CH - 1)) * 16;                 // (units are 16 rows or more apart: the same in each)
        lds = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char*)s_buf + wave * 1024;
    }
    // rows row0 .. row0 + ROWS - 1 to LDS from buffer `buf` on; rows past the end re-read the last token
    template <int ROWS = kRows>
    __device__ __forceinline__ void copy(int row0, int T, int buf) const
    {
        constexpr int units = ROWS / kUnitRows / WAVES;
        const char* from = base + (long)row0 * stride;
        const uint32_t to = lds + buf * kBufBytes;
        const uint32_t left = T - 1 - row0;                     // (row0 is a token)
        if (left >= ROWS - 1) {                                 // the same in every lane
            const uint32_t off = row * stride + chunk;
#pragma unroll
            for (int i = 0; i < units; i++) lds_copy16(from + (long)(i * WAVES * kUnitRows) * stride, off, to + i * WAVES * 1024);
        } else {
#pragma unroll
            for (int i = 0; i < units; i++)
                lds_copy16(from, min(row + i * WAVES * kUnitRows, left) * stride + chunk, to + i * WAVES * 1024);
        }
    }
};

template <int D>
__device__ __forceinline__ uint4 staged_piece(const char* frag, int ln, int kb, int c)
{
    const int ch = (c >> 1) * 4 + kb * 2 + (c & 1);
    return *reinterpret_cast<const uint4*>(frag + ln * (D * 2) + ((ch ^ (ln & (D / 8 - 1))) << 4));
}

// Workgroup -> (block of 64 OWNERS tokens, head) for the two kernels below.  An XCD gets whole heads, as above.  Under the
// causal mask a block's work grows (pass 1) or shrinks (pass 2) with its position: the longest blocks of all heads come
// first, so that what a compute unit gets when it has finished one is the shorter the later it is (LONG_LAST: the last block
// is the longest).
template <bool LONG_LAST>
__device__ __forceinline__ void block_and_head(int nblk, int n_heads, int& blk, int& head)
{
    const int lin = blockIdx.x + nblk * blockIdx.y;           // grid = nblk n_heads, or (nblk, n_heads) if that is too long
    int rank;
    if (n_heads % 8 == 0) {
        const int per = n_heads >> 3, xcd = lin & 7, j = lin >> 3;
        rank = j / per;
        head = xcd * per + (j - rank * per);
    } else {
        rank = lin / n_heads;
        head = lin - rank * n_heads;
    }
    blk = LONG_LAST ? nblk - 1 - rank : rank;
}

// The logits tiles of one staged fragment against the two register-held ones, and beside them the vector work on the fragment
// before: 32 values a lane, of which work(e, n) requests the exponentials of e .. e + n - 1 and uses those of the call before, so
// that nothing waits for a result it has just asked for.  The order is pinned by scheduling barriers: left to itself the
// compiler puts each LDS read right in front of its product and each exponential right in front of its use.
// KEYS_STAGED: the staged rows are the keys.
// 16-byte pieces requested from LDS ahead of their products (4096 x 32, unmasked, 2 / 3 / 4: d = 128 280 / 278 / 273 us, d = 64 203 / 204 / 207)
// (with four wavefronts a workgroup, three of which are to be resident: two)
template <int D, int WAVES>
constexpr int kAtAhead = (D == 128) ? 4 : (WAVES == 8) ? 3 : 2;

// in: the first AHEAD pieces, requested before; left with those of the fragment behind this one if MORE.
template <int D, bool KEYS_STAGED, bool MORE, int AHEAD, typename Work>
__device__ __forceinline__ void staged_tiles(const char* frag, int ln, int kb, const AtFrag<D> (&own)[2], uint4 (&in)[AHEAD],
                                             float16_t (&acc)[2], Work work)
{
    constexpr int N = D / 16, kEach = 32 / N;
    uint4 piece[N + AHEAD];
#pragma unroll
    for (int c = 0; c < AHEAD; c++) piece[c] = in[c];
#pragma unroll
    for (int o = 0; o < 2; o++)
#pragma unroll
        for (int i = 0; i < 16; i++) acc[o][i] = 0.0f;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int c = 0; c < N; c++) {
        if (c + AHEAD < N) piece[c + AHEAD] = staged_piece<D>(frag, ln, kb, c + AHEAD);
        else if (MORE) piece[c + AHEAD] = staged_piece<D>(frag + 32 * D * 2, ln, kb, c + AHEAD - N);
        const bf16x8_t staged = __builtin_bit_cast(bf16x8_t, piece[c]);
#pragma unroll
        for (int o = 0; o < 2; o++) {
            const bf16x8_t mine = __builtin_bit_cast(bf16x8_t, own[o].c[c]);
            acc[o] = KEYS_STAGED ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(staged, mine, acc[o], 0, 0, 0)
                                 : __builtin_amdgcn_mfma_f32_32x32x16_bf16(mine, staged, acc[o], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            work(c * kEach + o * (kEach / 2), std::integral_constant<int, kEach / 2>());
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if (MORE)
#pragma unroll
        for (int c = 0; c < AHEAD; c++) in[c] = piece[N + c];
}

// The wavefront's two fragments of the block's rows, through the buffers that hold no stage yet (a lane's own loads of them would
// touch 32 rows for 32 bytes each); start() starts the first stage's copies, which arrive with them.
template <int D, int OWNERS, int WAVES, typename Start>
__device__ __forceinline__ void own_fragments(const AtWide<D, OWNERS, WAVES>& st, int blk, int owner, const char* from, int ln, int kb, int T,
                                              AtFrag<D> (&own)[2], Start start)
{
    static_assert(OWNERS * 64 * D * 2 <= (AtWide<D, OWNERS, WAVES>::kBufs - 1) * AtWide<D, OWNERS, WAVES>::kBufBytes, "the block's rows fit behind the first stage");
    st.template copy<OWNERS * 64>(blk * OWNERS * 64, T, 1);
    start();
    wait_lds_copies<0>();
    __syncthreads();
#pragma unroll
    for (int o = 0; o < 2; o++)
#pragma unroll
        for (int c = 0; c < D / 16; c++) own[o].c[c] = staged_piece<D>(from + (owner * 2 + o) * (32 * D * 2), ln, kb, c);
    __syncthreads();                    // all have read theirs
}

// Pass 1, long sequences: a wavefront owns the queries of two fragments; keys stream through LDS.
// m is a reference for the exponents, not always the maximum: it is raised to the maximum seen only when a sum of sixteen
// exponentials exceeds kAtRaise (or is the first), so an argument exceeds m by 8 at most and the steady state needs neither
// maxima nor rescaling.
constexpr float kAtRaise = 256.0f;

template <int D, int OWNERS, int WAVES>
__global__ __launch_bounds__(WAVES * kWave, at_resident(D, WAVES) * WAVES / 4) void attn_rowstats_wide_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, int T, int n_heads, int group,
    float scale_log2, int causal, float2* __restrict__ stats)
{
    using Stage = AtWide<D, OWNERS, WAVES>;
    __shared__ __attribute__((aligned(16))) char s_buf[Stage::kBufs][Stage::kBufBytes];
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int ln = lane & 31, kb = lane >> 5;
    const int nfrag = (T + 31) >> 5;
    const int owner = wave % OWNERS, stream = wave / OWNERS;
    int blk, h;
    block_and_head<true>((nfrag + 2 * OWNERS - 1) / (2 * OWNERS), n_heads, blk, h);
    const uint16_t* qh = q + (long)h * D;
    const uint16_t* kh = k + (long)(h / group) * D;
    const int qf = 2 * (OWNERS * blk + owner);                  // and the fragment behind it
    const int kf_last = causal ? min(2 * OWNERS * (blk + 1), nfrag) - 1 : nfrag - 1;
    const int mine_last = (qf >= nfrag) ? -1 : causal ? min(qf + 1, nfrag - 1) : kf_last;     // the last fragment these queries see
    // the fragments before this one need no mask: all but the diagonal and a ragged last one
    const int plain_end = min(causal ? qf : nfrag, T >> 5);
    const Stage st(kh, n_heads / group, s_buf[0], wave, lane);
    AtFrag<D> fq[2];
    own_fragments<D, OWNERS, WAVES>(Stage(qh, n_heads, s_buf[0], wave, lane), blk, owner, s_buf[1], ln, kb, T, fq, [&] { st.copy(0, T, 0); });
    if (Stage::kBufs == 3 && Stage::kFrags <= kf_last) st.copy(Stage::kRows, T, 1);
    float m[2] = {kMasked, kMasked}, l[2] = {0.0f, 0.0f};
    float sum[4], last[8];                                      // sum[2 o], sum[2 o + 1]: query fragment o
    auto begin = [&] { sum[0] = sum[1] = sum[2] = sum[3] = 0.0f; };
    auto exps = [&](const float16_t (&acc)[2], int e, auto n) {
        constexpr int N = decltype(n)::value;
        float t[N];
#pragma unroll
        for (int j = 0; j < N; j++) t[j] = fmaf(acc[(e + j) >> 4][(e + j) & 15], scale_log2, -m[(e + j) >> 4]);
#pragma unroll
        for (int j = 0; j < N; j++) t[j] = __builtin_amdgcn_exp2f(t[j]);
#pragma unroll
        for (int j = 0; j < N; j++) {
            if (e > 0) sum[2 * ((e - N + j) >> 4) + (j & 1)] += last[j];
            last[j] = t[j];
        }
    };
    auto finish = [&](auto n) {
        constexpr int N = decltype(n)::value;
#pragma unroll
        for (int j = 0; j < N; j++) sum[2 + (j & 1)] += last[j];
        return make_float2(sum[0] + sum[1], sum[2] + sum[3]);
    };
    auto plain = [&](const float16_t (&acc)[2]) {
        begin();
#pragma unroll
        for (int e = 0; e < 32; e += 8) exps(acc, e, std::integral_constant<int, 8>());
        return finish(std::integral_constant<int, 8>());
    };
    auto take = [&](const float16_t (&acc)[2], float2 sum) {
        if (__builtin_expect(__any(fmaxf(sum.x, sum.y) > kAtRaise), 0)) {
#pragma unroll
            for (int o = 0; o < 2; o++) {
                // the scale is positive, so the maximum is taken over the raw logits
                float raw = acc[o][0];
#pragma unroll
                for (int i = 1; i < 16; i++) raw = fmaxf(raw, acc[o][i]);
                const float mx = fmaxf(m[o], raw * scale_log2);
                float add = 0.0f;
#pragma unroll
                for (int i = 0; i < 16; i++) add += __builtin_amdgcn_exp2f(fmaf(acc[o][i], scale_log2, -mx));
                l[o] = l[o] * __builtin_amdgcn_exp2f(m[o] - mx) + add;
                m[o] = mx;
            }
        } else {
            l[0] += sum.x;
            l[1] += sum.y;
        }
    };
    // One fragment's products beside the exponentials of the one before (fragment kp).
    auto hide = [&](float16_t (&acc)[2], int kf) {
        if (__builtin_expect(kf >= plain_end, 0)) {
#pragma unroll
            for (int o = 0; o < 2; o++) {
                // the last key this lane's query sees, counted from the lane's first key
                const int last = (causal ? min((qf + o) * 32 + ln, T - 1) : T - 1) - kf * 32 - 4 * kb;
#pragma unroll
                for (int i = 0; i < 16; i++) acc[o][i] = (8 * (i >> 2) + (i & 3) <= last) ? acc[o][i] : -INFINITY;
            }
        }
    };
    float16_t acc0[2], acc1[2];
#pragma unroll
    for (int o = 0; o < 2; o++)
#pragma unroll
        for (int i = 0; i < 16; i++) acc1[o][i] = -INFINITY;    // nothing before the first
    int kp = -1;
    uint4 in[kAtAhead<D, WAVES>];
    for (int base = 0, buf = 0; base <= kf_last; base += Stage::kFrags, buf = (buf == Stage::kBufs - 1) ? 0 : buf + 1) {
        constexpr int ahead = (Stage::kBufs - 1) * Stage::kFrags;
        const bool more = base + ahead <= kf_last;              // the same in every thread
        if (more) st.copy((base + ahead) * 32, T, (buf == 0) ? Stage::kBufs - 1 : buf - 1);
        const int kf = base + Stage::kEach * stream;
        const char* frag = s_buf[buf] + Stage::kEach * stream * Stage::kFragBytes;
        if (kf <= mine_last) {                                  // the same in every lane of the wavefront
#pragma unroll
            for (int c = 0; c < kAtAhead<D, WAVES>; c++) in[c] = staged_piece<D>(frag, ln, kb, c);
        }
#pragma unroll
        for (int f = 0; f < Stage::kEach; f++) {
            if (kf + f <= mine_last) {
                float16_t(&acc)[2] = (f & 1) ? acc1 : acc0;
                float16_t(&before)[2] = (f & 1) ? acc0 : acc1;
                hide(before, kp);
                begin();
                auto work = [&](int e, auto n) { exps(before, e, n); };
                if (f + 1 < Stage::kEach) staged_tiles<D, true, true>(frag + f * Stage::kFragBytes, ln, kb, fq, in, acc, work);
                else staged_tiles<D, true, false>(frag + f * Stage::kFragBytes, ln, kb, fq, in, acc, work);
                take(before, finish(std::integral_constant<int, D == 128 ? 2 : 4>()));
                kp = kf + f;
            }
        }
        if (Stage::kBufs == 3 && more) wait_lds_copies<Stage::kUnits>();        // the next stage is there, the one behind it on its way
        else wait_lds_copies<0>();
        __syncthreads();
    }
    if (kp & 1) {                                               // the last fragment's exponentials (odd where there is none, too)
        hide(acc1, kp);
        take(acc1, plain(acc1));
    } else {
        hide(acc0, kp);
        take(acc0, plain(acc0));
    }
    float2(*const s_ml)[OWNERS * 64] = reinterpret_cast<float2(*)[OWNERS * 64]>(s_buf);
#pragma unroll
    for (int o = 0; o < 2; o++) {
        const float m2 = __shfl_xor(m[o], 32, kWave), l2 = __shfl_xor(l[o], 32, kWave);
        const float M = fmaxf(m[o], m2);
        const float L = l[o] * __builtin_amdgcn_exp2f(m[o] - M) + l2 * __builtin_amdgcn_exp2f(m2 - M);
        if (kb == 0) s_ml[stream][owner * 64 + o * 32 + ln] = make_float2(M, L);
    }
    __syncthreads();
    const int query = blk * OWNERS * 64 + threadIdx.x;
    if (threadIdx.x < OWNERS * 64 && query < T) {
        float M = s_ml[0][threadIdx.x].x;
#pragma unroll
        for (int s = 1; s < Stage::kStreams; s++) M = fmaxf(M, s_ml[s][threadIdx.x].x);
        float L = 0.0f;
#pragma unroll
        for (int s = 0; s < Stage::kStreams; s++) L += s_ml[s][threadIdx.x].y * __builtin_amdgcn_exp2f(s_ml[s][threadIdx.x].x - M);
        stats[(long)h * T + query] = make_float2(M, 1.0f / L);
    }
}

// Pass 2, long sequences: a wavefront owns the keys of two fragments; queries stream through LDS.
template <int D, int OWNERS, int WAVES>
__global__ __launch_bounds__(WAVES * kWave, at_resident(D, WAVES) * WAVES / 4) void attn_colsum_wide_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, int T, int n_heads, int group,
    float scale_log2, int causal, const float2* __restrict__ stats, float* __restrict__ partial)
{
    using Stage = AtWide<D, OWNERS, WAVES>;
    __shared__ __attribute__((aligned(16))) char s_buf[Stage::kBufs][Stage::kBufBytes];
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int ln = lane & 31, kb = lane >> 5;
    const int nfrag = (T + 31) >> 5;
    const int owner = wave % OWNERS, stream = wave / OWNERS;
    int blk, h;
    block_and_head<false>((nfrag + 2 * OWNERS - 1) / (2 * OWNERS), n_heads, blk, h);
    const uint16_t* qh = q + (long)h * D;
    const uint16_t* kh = k + (long)(h / group) * D;
    const float2* sh = stats + (long)h * T;
    const int kf = 2 * (OWNERS * blk + owner);
    const int first = causal ? 2 * OWNERS * blk : 0;
    const int mine_first = (kf >= nfrag) ? nfrag : causal ? kf : 0;     // the first fragment of queries that see these keys
    const Stage st(qh, n_heads, s_buf[0], wave, lane);
    float2 next[Stage::kEach], now[Stage::kEach];               // (m, 1 / l) of the lane's query in the wavefront's fragments
    auto request = [&](int qf) {
#pragma unroll
        for (int s = 0; s < Stage::kEach; s++) next[s] = sh[min((qf + Stage::kEach * stream + s) * 32 + ln, T - 1)];
    };
    constexpr bool three = at_resident(D, WAVES) * WAVES == 12;  // wavefronts a SIMD: a trip ahead four registers spill, and the two others cover the wait
    if (!three) request(first);
    AtFrag<D> fk[2];
    own_fragments<D, OWNERS, WAVES>(Stage(kh, n_heads / group, s_buf[0], wave, lane), blk, owner, s_buf[1], ln, kb, T, fk,
                             [&] { st.copy(first * 32, T, 0); });
    if (Stage::kBufs == 3 && first + Stage::kFrags < nfrag) st.copy((first + Stage::kFrags) * 32, T, 1);
    float col[2][16];
#pragma unroll
    for (int o = 0; o < 2; o++)
#pragma unroll
        for (int i = 0; i < 16; i++) col[o][i] = 0.0f;
    // p = exp2(logit' - m) / l, the last factor with the addition
    float last[8];
    auto exps = [&](const float16_t (&acc)[2], float2 ml, int e, auto n) {
        constexpr int N = decltype(n)::value;
        float t[N];
#pragma unroll
        for (int j = 0; j < N; j++) t[j] = fmaf(acc[(e + j) >> 4][(e + j) & 15], scale_log2, -ml.x);
#pragma unroll
        for (int j = 0; j < N; j++) t[j] = __builtin_amdgcn_exp2f(t[j]);
#pragma unroll
        for (int j = 0; j < N; j++) {
            if (e > 0) col[(e - N + j) >> 4][(e - N + j) & 15] = fmaf(last[j], ml.y, col[(e - N + j) >> 4][(e - N + j) & 15]);
            last[j] = t[j];
        }
    };
    auto finish = [&](float2 ml, auto n) {
        constexpr int N = decltype(n)::value;
#pragma unroll
        for (int j = 0; j < N; j++) col[1][16 - N + j] = fmaf(last[j], ml.y, col[1][16 - N + j]);
    };
    // A fragment that the mask or the last query cuts is added here, and what the next products then find before them adds
    // nothing.  (Keys past the end are added to places of their own, which nothing reads.  What is masked adds zero whatever its
    // query's statistics are: a query that is not a number spoils the keys that it sees and no others.)
    auto cut = [&](float16_t (&acc)[2], float2& ml, int qf) {
        if (__builtin_expect((qf + 1) * 32 > T || (causal && qf <= kf + 1), 0)) {
            const int query = qf * 32 + ln;
            // the last key this lane's query adds to, counted from the lane's first key
            const int last = (query >= T || qf < 0) ? -1 : causal ? query - kf * 32 - 4 * kb : 64;
#pragma unroll
            for (int o = 0; o < 2; o++)
#pragma unroll
                for (int i = 0; i < 16; i++) {
                    float p = __builtin_amdgcn_exp2f(fmaf(acc[o][i], scale_log2, -ml.x)) * ml.y;
                    p = (32 * o + 8 * (i >> 2) + (i & 3) <= last) ? p : 0.0f;
                    col[o][i] += p;
                    acc[o][i] = -INFINITY;
                }
            ml = make_float2(0.0f, 0.0f);
        }
    };
    float16_t acc0[2], acc1[2];
#pragma unroll
    for (int o = 0; o < 2; o++)
#pragma unroll
        for (int i = 0; i < 16; i++) acc1[o][i] = -INFINITY;    // nothing before the first
    int qp = -1;
    uint4 in[kAtAhead<D, WAVES>];
    float2 ml = make_float2(0.0f, 0.0f);                        // what goes with the fragment before
    for (int base = first, buf = 0; base < nfrag; base += Stage::kFrags, buf = (buf == Stage::kBufs - 1) ? 0 : buf + 1) {
        constexpr int ahead = (Stage::kBufs - 1) * Stage::kFrags;
        const bool more = base + ahead < nfrag;                 // the same in every thread
        if (three) request(base);
#pragma unroll
        for (int s = 0; s < Stage::kEach; s++) now[s] = next[s];
        if (!three) request(base + Stage::kFrags);
        __builtin_amdgcn_sched_barrier(0);                      // ahead of the copies, which may still be on their way at the trip's end
        if (more) st.copy((base + ahead) * 32, T, (buf == 0) ? Stage::kBufs - 1 : buf - 1);
        const int qf = base + Stage::kEach * stream;
        const char* frag = s_buf[buf] + Stage::kEach * stream * Stage::kFragBytes;
#pragma unroll
        for (int f = 0; f < Stage::kEach; f++) {
            if (qf + f >= mine_first && qf + f < nfrag) {       // the same in every lane of the wavefront (mine_first is even)
                if (f == 0) {
#pragma unroll
                    for (int c = 0; c < kAtAhead<D, WAVES>; c++) in[c] = staged_piece<D>(frag + f * Stage::kFragBytes, ln, kb, c);
                }
                float16_t(&acc)[2] = (f & 1) ? acc1 : acc0;
                float16_t(&before)[2] = (f & 1) ? acc0 : acc1;
                cut(before, ml, qp);
                auto work = [&](int e, auto n) { exps(before, ml, e, n); };
                if (f + 1 < Stage::kEach) staged_tiles<D, false, true>(frag + f * Stage::kFragBytes, ln, kb, fk, in, acc, work);
                else staged_tiles<D, false, false>(frag + f * Stage::kFragBytes, ln, kb, fk, in, acc, work);
                finish(ml, std::integral_constant<int, D == 128 ? 2 : 4>());
                qp = qf + f;
                ml = now[f];
            }
        }
        if (Stage::kBufs == 3 && more) wait_lds_copies<Stage::kUnits>();        // the next stage is there, the one behind it on its way
        else wait_lds_copies<0>();
        __syncthreads();
    }
    auto rest = [&](float16_t (&acc)[2]) {                      // the last fragment's exponentials
        cut(acc, ml, qp);
#pragma unroll
        for (int e = 0; e < 32; e += 8) exps(acc, ml, e, std::integral_constant<int, 8>());
        finish(ml, std::integral_constant<int, 8>());
    };
    if (qp & 1) rest(acc1);                                     // (none at all: nothing before the first)
    else rest(acc0);
    // Sums over the 32 queries that the lanes of each half hold: in every exchange a lane keeps half of its keys, so that it ends with
    // one, number ln % 16 of the sixteen (bits reversed) ...
    float* const s_col = reinterpret_cast<float*>(s_buf);       // [stream][OWNERS * 64]
#pragma unroll
    for (int o = 0; o < 2; o++) {
        int mine = 0;
#pragma unroll
        for (int w = 8, bit = 1; w > 0; w >>= 1, bit <<= 1) {
            const bool upper = (ln & bit) != 0;
#pragma unroll
            for (int i = 0; i < 8; i++)
                if (i < w) {
                    const float keep = upper ? col[o][i + w] : col[o][i], give = upper ? col[o][i] : col[o][i + w];
                    col[o][i] = keep + __shfl_xor(give, bit, kWave);
                }
            mine += upper ? w : 0;
        }
        const float v = col[o][0] + __shfl_xor(col[o][0], 16, kWave);
        if (ln < 16) s_col[stream * (OWNERS * 64) + owner * 64 + o * 32 + tile_key(0, kb, mine)] = v;
    }
    __syncthreads();
    // ... and over the wavefronts that share the keys, in their order
    const int key = blk * OWNERS * 64 + threadIdx.x;
    if (threadIdx.x < OWNERS * 64 && key < T) {
        float v = s_col[threadIdx.x];
#pragma unroll
        for (int s = 1; s < Stage::kStreams; s++) v += s_col[s * (OWNERS * 64) + threadIdx.x];
        partial[(long)h * T + key] = v;
    }
}

// s[i] = (sum over heads, in head order) / (Hh T).  Bound: a memory latency per batch of heads, sixteen of them; the last
// batch asks for the last head again where it is not whole.  A wavefront per workgroup, so that 4096 tokens reach 64
// compute units.  The whole score, us, one head at a time and 256 tokens per workgroup / so: 4096 tokens x 32 heads 207 / 196,
// 200 x 32 18.0 / 12.3, 200 x 12 14.1 / 12.1, 200 x 4 12.2 / 11.8, 200 x 1 11.2 / 11.3 (d = 128, causal).
// This kernel alone in a trace of 4096 x 32: 10.6 -> 4.8 us.
constexpr int kAtScoreThreads = kWave;

__global__ __launch_bounds__(kAtScoreThreads) void attn_score_kernel(const float* __restrict__ partial, int T, int n_heads,
                                                         float inv, float* __restrict__ score)
{
    const int i = blockIdx.x * kAtScoreThreads + threadIdx.x;
    if (i >= T) return;
    float s = 0.0f;
    if (n_heads <= 2) {
        const float first = partial[i], last = partial[(long)(n_heads - 1) * T + i];
        s += first;
        if (n_heads == 2) s += last;
        score[i] = s * inv;                 // (ahead of the rest: the code of the batches is several cache lines long)
        return;
    }
    int h = 0;
    for (; h + 16 <= n_heads; h += 16) {
        float v[16];
#pragma unroll
        for (int u = 0; u < 16; u++) v[u] = partial[(long)(h + u) * T + i];
#pragma unroll
        for (int u = 0; u < 16; u++) s += v[u];
    }
    if (h < n_heads) {
        float v[16];
#pragma unroll
        for (int u = 0; u < 16; u++) v[u] = partial[(long)min(h + u, n_heads - 1) * T + i];
#pragma unroll
        for (int u = 0; u < 16; u++)
            if (h + u < n_heads) s += v[u];
    }
    score[i] = s * inv;
}

static size_t attn_stats_bytes(int T, int n_heads) { return ((size_t)T * n_heads * sizeof(float2) + 255) / 256 * 256; }

}  // namespace dymoe

extern "C" {

size_t dymoe_attention_workspace_bytes(int T, int n_heads)
{
    if (T <= 0 || n_heads <= 0) return 0;
    return dymoe::attn_stats_bytes(T, n_heads) + ((size_t)T * n_heads * sizeof(float) + 255) / 256 * 256;
}

int dymoe_token_score_attention(dymoe_ctx* ctx, const void* q, const void* k, int T, int n_heads,
                                int n_kv_heads, int head_dim, float scale, int causal, float* score,
                                void* workspace, size_t workspace_bytes, void* stream)
{
    DYMOE_REQUIRE(T >= 0 && n_heads > 0 && n_kv_heads > 0 && n_heads % n_kv_heads == 0);
    DYMOE_REQUIRE(head_dim > 0 && head_dim % 8 == 0);
    DYMOE_REQUIRE(scale >= 0.0f && (causal == 0 || causal == 1));
    if (T == 0) return ctx ? DYMOE_OK : DYMOE_ENOCTX;
    DYMOE_REQUIRE(q && k && score && workspace);
    DYMOE_REQUIRE(dymoe_aligned(q, 16) && dymoe_aligned(k, 16) && dymoe_aligned(score, 4) &&
                  dymoe_aligned(workspace, 256));
    if (head_dim != 64 && head_dim != 128) return DYMOE_ENOTSUP;
    if (n_heads > 65535) return DYMOE_ENOTSUP;
    if (workspace_bytes < dymoe_attention_workspace_bytes(T, n_heads)) return DYMOE_ENOSPC;
    if (!ctx) return DYMOE_ENOCTX;
    hipStream_t st = (hipStream_t)stream;
    const uint16_t* qb = (const uint16_t*)q;
    const uint16_t* kbp = (const uint16_t*)k;
    float2* stats = reinterpret_cast<float2*>(workspace);
    float* partial = reinterpret_cast<float*>((char*)workspace + dymoe::attn_stats_bytes(T, n_heads));
    const int group = n_heads / n_kv_heads;
    const float s = (scale > 0.0f) ? scale : 1.0f / sqrtf((float)head_dim);
    const float scale_log2 = s * 1.44269504088896340736f;
    const int nfrag = (T + 31) / 32;
    const dymoe::AtChoice choice = dymoe::attn_choice(nfrag, n_heads, causal, head_dim, ctx->num_cu);
    const int owners = choice.owners, waves = choice.waves;
    const bool wide = owners != 0;
    // A dimension of a launch holds fewer than 2^32 threads: beyond that (from 275 GB of queries on) a head per y, as in the
    // narrow pair's launches.
    const int nblk = wide ? (nfrag + 2 * owners - 1) / (2 * owners) : 0;
    const long blocks = (long)nblk * n_heads;
    const int threads = waves * dymoe::kWave;
    const dim3 grid = !wide ? dim3((unsigned)nfrag, (unsigned)n_heads)
                      : blocks * threads < 1L << 32 ? dim3((unsigned)blocks)
                                                              : dim3((unsigned)nblk, (unsigned)n_heads);
#define DYMOE_ATTN_PAIR(STATS_, COLSUM_)                                                                               \
    do {                                                                                                               \
        dymoe_launch(ctx, DYMOE_K_ATTN_STATS, STATS_, grid, dim3(threads), 0, st, qb, kbp, T, n_heads, group,            \
                     scale_log2, causal, stats);                                                                       \
        DYMOE_HIP_LAUNCH_CHECK();                                                                                      \
        dymoe_launch(ctx, DYMOE_K_ATTN_COLSUM, COLSUM_, grid, dim3(threads), 0, st, qb, kbp, T, n_heads, group,          \
                     scale_log2, causal, (const float2*)stats, partial);                                               \
    } while (0)
#define DYMOE_ATTN_WIDE(D_, OWNERS_, WAVES_) \
    DYMOE_ATTN_PAIR((dymoe::attn_rowstats_wide_kernel<D_, OWNERS_, WAVES_>), (dymoe::attn_colsum_wide_kernel<D_, OWNERS_, WAVES_>))
    if (head_dim == 128) {
        if (owners == 2 && waves == 4) DYMOE_ATTN_WIDE(128, 2, 4);
        else if (owners == 4) DYMOE_ATTN_WIDE(128, 4, 8);
        else if (owners == 2) DYMOE_ATTN_WIDE(128, 2, 8);
        else DYMOE_ATTN_PAIR(dymoe::attn_rowstats_kernel<128>, dymoe::attn_colsum_kernel<128>);
    } else {
        if (owners == 2 && waves == 4) DYMOE_ATTN_WIDE(64, 2, 4);
        else if (owners == 2) DYMOE_ATTN_WIDE(64, 2, 8);
        else DYMOE_ATTN_PAIR(dymoe::attn_rowstats_kernel<64>, dymoe::attn_colsum_kernel<64>);
    }
#undef DYMOE_ATTN_WIDE
#undef DYMOE_ATTN_PAIR
    DYMOE_HIP_LAUNCH_CHECK();
    hipLaunchKernelGGL(dymoe::attn_score_kernel, dim3((unsigned)((T + dymoe::kAtScoreThreads - 1) / dymoe::kAtScoreThreads)),
                       dim3(dymoe::kAtScoreThreads), 0, st,
                       (const float*)partial, T, n_heads, 1.0f / ((float)n_heads * (float)T), score);
    DYMOE_HIP_LAUNCH_CHECK();
    return DYMOE_OK;
}

}  // extern "C"
