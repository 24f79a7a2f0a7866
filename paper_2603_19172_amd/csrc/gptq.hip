// Error-compensated quantize-and-pack (paper Sec. 5: GPTQ is the base quantizer
// of the paper's implementation).  Same outputs as the plain quantizer (codes,
// fp16 scale and zero per group of 64 columns, row-major), but a row is
// quantised column by column and what rounding takes away from column c is
// spread over the columns still to come, so that the layer's output on the
// calibration inputs changes least:
//     e = (v[c] - dequant(q_c)) / U[c,c],    v[j] = fma(-e, U[c,j], v[j])  for j > c,
// U the upper triangular factor of the inverse of the (damped) Hessian
// H = X^T X of the calibration inputs, H^-1 = U^T U.  Scale and zero of a group
// are taken from the row's corrected values when the group is reached.
//
// The arithmetic is an exact sequence of binary32 operations, columns in
// ascending order, one fused multiply-add per correction (this file is built
// with -ffp-contract=off, the fma is written out): the codes must equal the
// reference's bit for bit, so the corrections may not be regrouped.
//
// The fp32 matrix instructions of this chip do not regroup them: v_mfma_f32_{16x16x4,32x32x2}_f32 give, bit for bit,
// what one fma after the other over ascending k gives, subnormals included (compared on 14 million random results with
// equal, cancelling, tiny and subnormal operands; the tests sweep rows against the plain chain as well).  So the
// corrections go through the matrix cores and keep the reference's bits: a register-only loop of those instructions holds
// 140 to 155 TFLOP/s on random data, one of vector fmas 108 to 117, and a lane's operands serve four times the products.
//
// Rows are independent, columns are not.  Columns go in panels of 256 (four groups of 64), two launches each:
//   group kernel   a wavefront owns 16 rows through the whole panel: a group's values lose the corrections of the
//                  panel's earlier groups (16x16x4 products, errors from LDS), are turned round so that four lanes
//                  share a row (a lane every fourth column), and are quantised column by column; codes, scale, zero
//                  and the errors e of the row are written;
//   trail kernel   v[:, j] for the columns behind the panel: 256 chained fmas per element.
// The working copy v of the matrix (fp32) lives in the caller's workspace.
#include <type_traits>

#include "common.hpp"

namespace dymoe {

constexpr int kGqGroup = 64;        // columns per group
constexpr int kGqRows = 64;         // rows per row block
constexpr int kGqPanel = 4;         // groups per panel
constexpr int kGqChunk = 16;        // columns per piece of a group's chain

typedef float f32x4_t __attribute__((ext_vector_type(4)));

static inline size_t gq_round256(size_t v) { return (v + 255) & ~(size_t)255; }
static inline long gq_row_blocks(long N) { return (N + kGqRows - 1) / kGqRows; }

// Groups per panel.  Where all rows make one ragged block, no block can keep its errors in v (see GqErr), and half a panel
// is kept in the linear buffer.
static inline int gq_panel(long N) { return (N < kGqRows) ? kGqPanel / 2 : kGqPanel; }

// bytes of the ragged row block's errors, a panel's columns of 64 rows; no ragged block, no buffer
static inline size_t gq_tail_bytes(long N) { return (N % kGqRows) ? (size_t)gq_panel(N) * kGqGroup * kGqRows * sizeof(float) : 0; }

// Where the (negated) errors of a panel of four groups are kept between the two kernels.  The panel's own columns of
// v are dead once its values are in registers, and a row block's 64 x 256 of them hold its 256 x 64 errors exactly:
// element (column c of the panel, row r of the block) sits in row c / 4 of the block at offset (c % 4) * 64 + r.  The
// ragged last row block has too few rows for that and uses a linear buffer of the same arrangement (row stride 256).
struct GqErr {
    float* whole;     // v + first column of the panel
    long ld;          // row stride of v
    float* tail;      // linear buffer of the ragged block
    long full_blocks;
};
__device__ __forceinline__ float* gq_err_block(const GqErr& g, long block, long& ld)
{
    const bool full = block < g.full_blocks;
    ld = full ? g.ld : 256;
    return full ? g.whole + block * kGqRows * g.ld : g.tail;
}

// x of column C, held by lane C % 4 of a quad in register C / 4, to the quad's four lanes
template <int Q>
__device__ __forceinline__ float quad_bcast(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), Q * 0x55, 0xF, 0xF, true));
}

// The two values a step of the column chain needs from the diagonal block of U besides its row: 1 / U[c,c] in 64 bits
// and U[c,c].  e = rest / U[c,c] is taken as (float)((double)rest * (1 / U)): the product is within 2^-52 of the
// quotient, and a quotient of two 24-bit numbers that is not itself halfway between two floats is at least 2^-49 away
// from it, so the rounding to float is the quotient's own, in 3 dependent instructions instead of the dozen of an IEEE
// division.  Halfway cases only exist among subnormal quotients: those are recognised and the group is done again with
// the division itself.
// One call does 16 columns, T0 .. T0 + 15 of the group: x[i] is column T0 + 4 i + q; what their errors do to the group's later
// columns is the caller's.
template <int BITS, int T0, typename Emit>
__device__ __forceinline__ bool gq_chunk_chain(float (&x)[4], int q, float m, float s, float inv, const float* s_d,
                                               const double* s_inv, uint32_t* words, Emit emit)
{
#pragma clang fp contract(off)
    constexpr int qmax = (1 << BITS) - 1;
    constexpr int per_word = 32 / BITS;
    bool subnormal = false;
    float keep = 0.0f;
    // the rows of the diagonal block (the lane's four columns), two steps' worth at a time, one batch ahead of their use: the
    // scheduling barriers keep the compiler from fetching each row only when it is needed
    float4 d[2][2];
    double rcp[2][2];
    auto fetch = [&](int b) {
#pragma unroll
        for (int c = 0; c < 2; c++) {
            rcp[b & 1][c] = s_inv[T0 + 2 * b + c];
            d[b & 1][c] = *reinterpret_cast<const float4*>(s_d + (T0 + 2 * b + c) * kGqChunk + 4 * q);
        }
    };
    fetch(0);
#pragma unroll
    for (int b = 0; b < kGqChunk / 2; b++) {
        __builtin_amdgcn_sched_barrier(0);
        if (b + 1 < kGqChunk / 2) fetch(b + 1);
        __builtin_amdgcn_sched_barrier(0);
        const int k = b / 2;
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int i = 2 * b + h, c = i & 3, at = T0 + i;
            const float xi = c == 0 ? quad_bcast<0>(x[k]) : c == 1 ? quad_bcast<1>(x[k]) : c == 2 ? quad_bcast<2>(x[k]) : quad_bcast<3>(x[k]);
            const float t = xi - m;
            float r = __builtin_rintf(t * inv);
            r = fminf(fmaxf(r, 0.0f), (float)qmax);
            if (at % per_word == 0) words[at / per_word] = 0u;
            words[at / per_word] |= (uint32_t)(int)r << (BITS * (at % per_word));
            float dq = r * s;
            dq = dq + m;
            const float rest = xi - dq;
            const float e = (float)((double)rest * rcp[b & 1][h]);
            subnormal |= __builtin_amdgcn_classf(e, 0x90);
            const float ne = -e;
            keep = (q == c) ? ne : keep;
            // (columns of register k that are already done change too; nothing reads them any more)
            const float dd[4] = {d[b & 1][h].x, d[b & 1][h].y, d[b & 1][h].z, d[b & 1][h].w};
#pragma unroll
            for (int j = (c == 3) ? k + 1 : k; j < 4; j++) x[j] = __builtin_fmaf(ne, dd[j], x[j]);
        }
        if (b & 1) emit(T0 / 4 + k, keep);
    }
    return subnormal;
}

// A whole group with the division itself, for rows with subnormal quotients: rare, so rolled up and in LDS (sx: the
// wavefront's 16 x 64 values, overwritten), the rows of U (ud: its diagonal block, row stride K) from memory.
template <int BITS, typename Emit>
__device__ __forceinline__ void gq_group_chain_exact(float* sx, int r, int q, float m, float s, float inv, const float* __restrict__ ud,
                                                     long K, uint32_t* words, Emit emit)
{
#pragma clang fp contract(off)
    constexpr int qmax = (1 << BITS) - 1;
    constexpr int per_word = 32 / BITS;
    float* const row = sx + r * (kGqGroup + 4);
    float keep = 0.0f;
#pragma unroll 1
    for (int i = 0; i < kGqGroup; i++) {
        const float xi = row[i];
        float t = (xi - m) * inv;
        t = fminf(fmaxf(__builtin_rintf(t), 0.0f), (float)qmax);
        float dq = t * s;
        dq = dq + m;
        const float ne = -((xi - dq) / ud[(long)i * K + i]);
        keep = (q == (i & 3)) ? ne : keep;
        if ((i & 3) == 3) emit(i >> 2, keep);
        for (int j = (i & ~3) + q; j < kGqGroup; j += 4)
            if (j > i) row[j] = __builtin_fmaf(ne, ud[(long)i * K + j], row[j]);
        if (q == (i & 3)) row[i] = t;                           // the code, in the place of the value
    }
#pragma unroll
    for (int i = 0; i < kGqGroup; i++) {
        if (i % per_word == 0) words[i / per_word] = 0u;
        words[i / per_word] |= (uint32_t)(int)row[i] << (BITS * (i % per_word));
    }
}

// One panel of up to four groups: rows in blocks of 64 (a workgroup), 16 rows a wavefront.  FIRST: the values come from
// the bf16 matrix itself (nothing has been corrected yet), so the working copy is never filled by a pass of its own.
// Bound: the chain of 64 dependent quantise-and-correct steps per group, 52 ns each, and the products between groups.  Four
// lanes share a row, so that 896 wavefronts work on the chip's 1024 SIMDs for 14336 rows; the chain corrects 16 columns only
// (four a lane: as few as its own latency covers, and a quarter of the reads of U from LDS), the group's later columns get
// those 16 errors as matrix products.  14336 x 4096, int4: 31 us per panel (2 to start, 4.5 per group, 8.6 between the groups);
// with the chain correcting all 64 columns 40 us, with a lane per row 120.
template <int BITS, bool FIRST>
__global__ __launch_bounds__(256) void gptq_group_kernel(
    const uint16_t* __restrict__ w, float* v, const float* __restrict__ u, long N, long K, long base,
    int n_groups, GqErr err, uint8_t* __restrict__ codes, uint16_t* __restrict__ scale, uint16_t* __restrict__ zero)
{
#pragma clang fp contract(off)
    constexpr int qmax = (1 << BITS) - 1;
    constexpr int n_words = kGqGroup * BITS / 32;               // 16 (int8), 8 (int4), 4 (int2)
    constexpr int kStride = kGqGroup + 4;
    __shared__ __attribute__((aligned(16))) float s_d[kGqPanel][kGqGroup * kGqChunk];   // the 16 x 16 diagonal blocks, [c][j % 4][j / 4]
    __shared__ __attribute__((aligned(16))) double s_inv[kGqPanel * kGqGroup];
    __shared__ __attribute__((aligned(16))) float s_e[4][kGqPanel * kGqGroup * 16];   // per wavefront [column][row], negated
    __shared__ __attribute__((aligned(16))) float s_x[4][16 * kStride];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const long row0 = (long)blockIdx.x * kGqRows + 16 * wave;
    // matrix-instruction layout: this lane holds rows 4 rg .. 4 rg + 3, columns 4 cl .. 4 cl + 3 of the 16 x 64 values
    const int rg = lane >> 4, cl = lane & 15;
    float4 cur[kGqPanel][4];
#pragma unroll
    for (int g = 0; g < kGqPanel; g++) {
        if (g >= n_groups) break;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const long row = min(row0 + 4 * rg + i, N - 1);     // rows past the last one redo it and keep the result to themselves
            const long at = row * K + base + kGqGroup * g + 4 * cl;
            if constexpr (FIRST) {
                const uint2 raw = load_global<uint2>(w + at);
                cur[g][i] = make_float4(bf16_lo(raw.x), bf16_hi(raw.x), bf16_lo(raw.y), bf16_hi(raw.y));
            } else {
                cur[g][i] = *reinterpret_cast<const float4*>(v + at);
            }
        }
    }
    for (int at = tid; at < n_groups * kGqGroup; at += 256) {
        const long c = base + at;
        s_inv[at] = 1.0 / (double)u[c * K + c];
    }
    for (int at = tid; at < n_groups * kGqGroup * 4; at += 256) {
        const int g = at >> 8, c = (at >> 2) & 63, i = at & 3;
        const float4 d = *reinterpret_cast<const float4*>(u + (base + kGqGroup * g + c) * K + base + kGqGroup * g + (c & ~15) + 4 * i);
        float* dst = &s_d[g][c * kGqChunk + i];
        dst[0] = d.x; dst[4] = d.y; dst[8] = d.z; dst[12] = d.w;
    }
    __syncthreads();            // and every wavefront has its values in registers: v may now be overwritten by errors
    const int r = lane >> 2, q = lane & 3;                      // the chain's layout: row r, columns 4 m + q
    const long row = row0 + r;
    long eld;
    float* const eb = gq_err_block(err, blockIdx.x, eld) + q * kGqRows + 16 * wave + r;
    // The rows of U that a group's values are corrected with come straight from memory, 32 columns ahead of their use; the
    // first batch of the next group is requested before this group's chain and lies in registers behind it.
    constexpr int kAhead = 8;
    float4 ub[2][kAhead];
    const float* bp = u + (base + rg) * K + base + kGqGroup + 4 * cl;
    auto fetch = [&](int buf, const float* from) {
#pragma unroll
        for (int i = 0; i < kAhead; i++) ub[buf][i] = load_global<float4>(from + (long)i * 4 * K);
        __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll 1
    for (int g = 0; g < n_groups; g++) {
        if (g > 0) {
            // the group's values move to the front (a run-time index would put them into private memory)
#pragma unroll
            for (int o = 1; o < kGqPanel; o++)
#pragma unroll
                for (int i = 0; i < 4; i++) cur[o - 1][i] = cur[o][i];
            f32x4_t acc[4];
#pragma unroll
            for (int i = 0; i < 4; i++) {
                acc[0][i] = cur[0][i].x; acc[1][i] = cur[0][i].y; acc[2][i] = cur[0][i].z; acc[3][i] = cur[0][i].w;
            }
            const float* ap = &s_e[wave][lane];
            auto multiply = [&](int buf) {
#pragma unroll
                for (int i = 0; i < kAhead; i++) {
                    const float a = ap[i * 64];
                    acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, ub[buf][i].x, acc[0], 0, 0, 0);
                    acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, ub[buf][i].y, acc[1], 0, 0, 0);
                    acc[2] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, ub[buf][i].z, acc[2], 0, 0, 0);
                    acc[3] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, ub[buf][i].w, acc[3], 0, 0, 0);
                }
                ap += kAhead * 64;
                __builtin_amdgcn_sched_barrier(0);
            };
            const float* from = bp;
#pragma unroll 1
            for (int h = 1; h < g; h++) {                       // a group's 64 columns are two batches
                fetch(1, from + (long)kAhead * 4 * K);
                multiply(0);
                from += (long)2 * kAhead * 4 * K;
                fetch(0, from);
                multiply(1);
            }
            fetch(1, from + (long)kAhead * 4 * K);
            multiply(0);
            multiply(1);
            bp += kGqGroup;
#pragma unroll
            for (int i = 0; i < 4; i++) cur[0][i] = make_float4(acc[0][i], acc[1][i], acc[2][i], acc[3][i]);
        }
        if (g + 1 < n_groups) fetch(0, bp);
        // U between the group's pieces of 16 columns: rows 16 t + 4 kk + rg, columns 16 tt + cl, tt > t
        float between[24];
        const float* const ud = u + (base + kGqGroup * g) * K + base + kGqGroup * g;
        {
            int n = 0;
#pragma unroll
            for (int t = 0; t < 3; t++)
#pragma unroll
                for (int tt = t + 1; tt < 4; tt++)
#pragma unroll
                    for (int kk = 0; kk < 4; kk++) between[n++] = load_global<float>(ud + (long)(16 * t + 4 * kk + rg) * K + 16 * tt + cl);
            __builtin_amdgcn_sched_barrier(0);
        }
        float* const sx = s_x[wave];                            // one wavefront's own: no barrier
#pragma unroll
        for (int i = 0; i < 4; i++) *reinterpret_cast<float4*>(&sx[(4 * rg + i) * kStride + 4 * cl]) = cur[0][i];
        float x[16];
#pragma unroll
        for (int m = 0; m < 16; m++) x[m] = sx[r * kStride + 4 * m + q];
        f32x4_t later[3];                                       // the pieces behind the first, in the matrix instructions' layout
#pragma unroll
        for (int tt = 1; tt < 4; tt++)
#pragma unroll
            for (int i = 0; i < 4; i++) later[tt - 1][i] = sx[(4 * rg + i) * kStride + 16 * tt + cl];
        float lo = x[0], hi = x[0];
#pragma unroll
        for (int m = 1; m < 16; m++) {
            lo = fminf(lo, x[m]);
            hi = fmaxf(hi, x[m]);
        }
        lo = fminf(lo, dpp_get<0xB1, 0xF>(lo));
        hi = fmaxf(hi, dpp_get<0xB1, 0xF>(hi));
        lo = fminf(lo, dpp_get<0x4E, 0xF>(lo));
        hi = fmaxf(hi, dpp_get<0x4E, 0xF>(hi));
        const _Float16 zh = (_Float16)lo;                       // round to nearest even
        const float range = hi - lo;
        const float step = range / (float)qmax;                 // correctly rounded division
        const _Float16 sh = (_Float16)step;
        const float m = (float)zh, s = (float)sh;
        const float inv = (s > 0.0f) ? (1.0f / s) : 0.0f;
        uint32_t words[n_words];
        float* const se = &s_e[wave][g * kGqGroup * 16 + q * 16 + r];
        auto emit = [&](int k, float ne) {                      // the errors of columns 4 k .. 4 k + 3, this lane's 4 k + q
            se[k * 64] = ne;
            eb[(long)(16 * g + k) * eld] = ne;                  // (unread behind the last panel; the place is dead all the same)
        };
        // Sixteen columns by the chain, then their products onto the pieces behind them, errors ascending as the chain would
        // have applied them.
        float piece[4] = {x[0], x[1], x[2], x[3]};
        const double* const si = &s_inv[g * kGqGroup];
        auto carry = [&](auto from) {
            constexpr int T = decltype(from)::value, first = T == 0 ? 0 : T == 1 ? 12 : 20;
            const float* const ap = &s_e[wave][(g * kGqGroup + 16 * T) * 16 + lane];
            float a[4];
#pragma unroll
            for (int kk = 0; kk < 4; kk++) a[kk] = ap[kk * 64];
#pragma unroll
            for (int tt = T + 1; tt < 4; tt++) {
#pragma unroll
                for (int kk = 0; kk < 4; kk++)
                    later[tt - 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[kk], between[first + 4 * (tt - T - 1) + kk], later[tt - 1], 0, 0, 0);
                if (tt == T + 1) {
#pragma unroll
                    for (int i = 0; i < 4; i++) sx[(4 * rg + i) * kStride + 16 * tt + cl] = later[tt - 1][i];
#pragma unroll
                    for (int i = 0; i < 4; i++) piece[i] = sx[r * kStride + 16 * tt + 4 * i + q];
                }
            }
        };
        bool subnormal = gq_chunk_chain<BITS, 0>(piece, q, m, s, inv, s_d[g], si, words, emit);
        carry(std::integral_constant<int, 0>());
        subnormal |= gq_chunk_chain<BITS, 16>(piece, q, m, s, inv, s_d[g], si, words, emit);
        carry(std::integral_constant<int, 1>());
        subnormal |= gq_chunk_chain<BITS, 32>(piece, q, m, s, inv, s_d[g], si, words, emit);
        carry(std::integral_constant<int, 2>());
        subnormal |= gq_chunk_chain<BITS, 48>(piece, q, m, s, inv, s_d[g], si, words, emit);
        if (__any(subnormal)) {
#pragma unroll
            for (int i = 0; i < 4; i++) *reinterpret_cast<float4*>(&sx[(4 * rg + i) * kStride + 4 * cl]) = cur[0][i];
            gq_group_chain_exact<BITS>(sx, r, q, m, s, inv, ud, K, words, emit);
        }
        if (row < N) {
            uint8_t* dst = codes + (row * K + base + kGqGroup * g) * BITS / 8;
            constexpr int mine = n_words / 4;                   // each lane of a quad writes a quarter of the row's codes
            uint32_t out[mine];
#pragma unroll
            for (int k = 0; k < mine; k++)
                out[k] = (q & 2) ? ((q & 1) ? words[3 * mine + k] : words[2 * mine + k]) : ((q & 1) ? words[mine + k] : words[k]);
            if constexpr (mine == 4) store_global(dst + 16 * q, make_uint4(out[0], out[1], out[2], out[3]));
            else if constexpr (mine == 2) store_global(dst + 8 * q, make_uint2(out[0], out[1]));
            else store_global(dst + 4 * q, out[0]);
            const long sg = row * (K / kGqGroup) + base / kGqGroup + g;
            if (q == 0) store_global(scale + sg, (uint16_t)f16_bits(sh));
            if (q == 1) store_global(zero + sg, (uint16_t)f16_bits(zh));
        }
    }
}

// 64 x 64 values in the layout of 4 x 4 tiles of v_mfma_f32_16x16x4_f32 whose rows and columns are interleaved: tile (a, b)
// register i of lane (rg = lane / 16, cl = lane % 16) is row 16 rg + 4 i + a, column 4 cl + b.  So a lane's operands for
// four tiles are four neighbouring floats, its 64 values are 16 rows of four neighbouring floats, and every load and
// store moves 16 bytes per lane, 256 bytes per row.
struct GqTile {
    f32x4_t t[4][4];
};

// acc += sum over c of A[c, row] B[c, column], c ascending, n a multiple of 16, for the 2 x 2 tiles of a workgroup (wavefront
// w: rows of tile row w / 2, columns of tile column w % 2).  Sixteen c's at a time go through LDS, fetched one stage
// (2048 cycles of products per wavefront) before they are stored there: a wavefront that streams its own operands
// from L2 twice as far ahead was bound by that traffic (85 TFLOP/s: the 32 KB of L1 hold no two wavefronts' batches).
// ap, bp: this wavefront's share of the operands, tile w % 2 and the c's 4 (w / 2) .. + 3 and 8 + 4 (w / 2) .. + 3 of a stage, at the
// lane's own place (c = rg, row or column 4 cl); lda4, ldb4: four c's further.
__device__ __forceinline__ void gq_tile_products(GqTile& acc, float* s_op, int wave, const float* ap, long lda4, const float* bp, long ldb4, int n)
{
    constexpr int kStage = 2 * 16 * kGqGroup;                   // floats of one operand
    const int lane = threadIdx.x & 63;
    float* const put = s_op + (wave & 1) * 16 * kGqGroup + (wave >> 1) * 4 * kGqGroup + 4 * lane;
    const float* const get_a = s_op + (wave >> 1) * 16 * kGqGroup + 4 * lane;
    const float* const get_b = s_op + kStage + (wave & 1) * 16 * kGqGroup + 4 * lane;
    float4 fa[2], fb[2];
    auto fetch = [&] {
        fa[0] = load_global<float4>(ap);
        fa[1] = load_global<float4>(ap + 2 * lda4);
        fb[0] = load_global<float4>(bp);
        fb[1] = load_global<float4>(bp + 2 * ldb4);
        ap += 4 * lda4;
        bp += 4 * ldb4;
        __builtin_amdgcn_sched_barrier(0);                      // or they move down to their use
    };
    auto park = [&](int buf) {
        float* const at = put + buf * 2 * kStage;
        *reinterpret_cast<float4*>(at) = fa[0];
        *reinterpret_cast<float4*>(at + 8 * kGqGroup) = fa[1];
        *reinterpret_cast<float4*>(at + kStage) = fb[0];
        *reinterpret_cast<float4*>(at + kStage + 8 * kGqGroup) = fb[1];
        __syncthreads();
    };
    auto multiply = [&](int buf) {
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const float4 av = *reinterpret_cast<const float4*>(get_a + buf * 2 * kStage + k * 4 * kGqGroup);
            const float4 bv = *reinterpret_cast<const float4*>(get_b + buf * 2 * kStage + k * 4 * kGqGroup);
            const float ar[4] = {av.x, av.y, av.z, av.w};
            const float br[4] = {bv.x, bv.y, bv.z, bv.w};
#pragma unroll
            for (int x = 0; x < 4; x++)
#pragma unroll
                for (int y = 0; y < 4; y++) acc.t[x][y] = __builtin_amdgcn_mfma_f32_16x16x4f32(ar[x], br[y], acc.t[x][y], 0, 0, 0);
        }
    };
    fetch();
    park(0);
    int buf = 0;
#pragma unroll 1
    for (int c = 16; c < n; c += 16) {
        fetch();
        multiply(buf);
        buf ^= 1;
        park(buf);              // this buffer's last readers passed the barrier of the stage before
    }
    multiply(buf);
}

// v[r, j] = fma(-E[c, r], U[c, j], v[r, j]) for the panel's n_cols columns c in ascending order, every row r, columns
// [col_begin, K).  A wavefront owns 64 x 64 values, a workgroup 128 x 128; FIRST: v's values are still those of w.
// Bound: fp32 matrix instructions (a register-only loop holds 150 TFLOP/s).  14336 rows, 256 columns over the 3840 behind
// them: 250 us = 113 TFLOP/s, and v is passed over 16 times for 4096 columns; as vector fmas, 128 columns a pass, the
// same corrections took 3.9 ms per matrix at 57 TFLOP/s where these take 2.1 ms.
template <bool FIRST>
__global__ __launch_bounds__(256, 2) void gptq_trail_kernel(const uint16_t* __restrict__ w, float* v, const float* __restrict__ u,
                                                         long N, long K, long base, int n_cols, long col_begin, GqErr err)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rg = lane >> 4, cl = lane & 15;
    // Workgroups are dealt to the eight XCDs in turn: an XCD takes every eighth pair of row blocks, and walks them eight
    // pairs at a time across all columns, so that the 64 tiles it runs at a time share 8 row and 8 column operands in its L2.
    const uint32_t row_pairs = (uint32_t)((N + 2 * kGqRows - 1) / (2 * kGqRows));
    const uint32_t col_pairs = (uint32_t)((K - col_begin + 2 * kGqGroup - 1) / (2 * kGqGroup));
    const uint32_t xcd = blockIdx.x & 7, at = blockIdx.x >> 3;
    const uint32_t per_xcd = (row_pairs + 7) >> 3;
    const uint32_t band = at / (8 * col_pairs), in_band = at - band * 8 * col_pairs;
    const uint32_t height = min(8u, per_xcd - 8 * band);
    const uint32_t cp = in_band / height, rp = xcd + 8 * (8 * band + in_band - cp * height);
    if (rp >= row_pairs) return;
    // a wavefront whose block lies outside (an odd number of blocks) works on the last one as well and keeps it to itself
    const long n_blocks = (N + kGqRows - 1) / kGqRows;
    const long block = min(2 * (long)rp + (wave >> 1), n_blocks - 1);
    const long col0 = min(col_begin + (2 * (long)cp + (wave & 1)) * kGqGroup, K - kGqGroup);
    const bool mine = 2 * (long)rp + (wave >> 1) == block && col_begin + (2 * (long)cp + (wave & 1)) * kGqGroup == col0;
    const long row0 = block * kGqRows;
    const bool whole = row0 + kGqRows <= N;
    __shared__ __attribute__((aligned(16))) float s_op[2 * 2 * 2 * 16 * kGqGroup];
    const uint32_t off = 16 * rg * (uint32_t)K + 4 * cl;
    GqTile acc;
    auto load = [&](int i, int a, const void* at) {
        float4 val;
        if constexpr (FIRST) {
            const uint2 raw = load_global<uint2>(at);
            val = make_float4(bf16_lo(raw.x), bf16_hi(raw.x), bf16_lo(raw.y), bf16_hi(raw.y));
        } else {
            val = load_global<float4>(at);
        }
        acc.t[a][0][i] = val.x; acc.t[a][1][i] = val.y; acc.t[a][2][i] = val.z; acc.t[a][3][i] = val.w;
    };
    const auto* src = [&] {
        if constexpr (FIRST) return w + row0 * K + col0;
        else return (const float*)v + row0 * K + col0;
    }();
    if (whole) {
#pragma unroll
        for (int r = 0; r < 16; r++) load(r >> 2, r & 3, src + r * K + off);
    } else {
        const int last = (int)(N - 1 - row0);
#pragma unroll
        for (int r = 0; r < 16; r++) load(r >> 2, r & 3, src + min(16 * rg + r, last) * K + 4 * cl);
    }
    long eld;
    const float* const eb = gq_err_block(err, min(2 * (long)rp + (wave & 1), n_blocks - 1), eld);
    gq_tile_products(acc, s_op, wave, eb + (wave >> 1) * eld + 4 * lane, eld, u + (base + 4 * (wave >> 1) + rg) * K + col0 + 4 * cl,
                            4 * K, n_cols);
    if (!mine) return;
    float* dst = v + row0 * K + col0;
    asm("" : "+s"(dst));        // the loads' 16 addresses are worked out again here, not kept through the products
    auto store = [&](int r) {
        const int i = r >> 2, a = r & 3;
        store_global(dst + r * K + off, make_float4(acc.t[a][0][i], acc.t[a][1][i], acc.t[a][2][i], acc.t[a][3][i]));
    };
    if (whole) {
#pragma unroll
        for (int r = 0; r < 16; r++) store(r);
    } else {
        const int rows = (int)(N - row0);
#pragma unroll
        for (int r = 0; r < 16; r++)
            if (16 * rg + r < rows) store(r);
    }
}

// The same corrections for launches that the kernel above leaves the chip half empty in (its workgroup takes 15 us of matrix
// instructions whatever there is beside it): a workgroup 64 x 64, a wavefront 32 x 32, the operands of 64 columns c at a time
// through LDS.  Up to three quarters of a workgroup of the other kernel per compute unit; a whole sweep, us, other / this:
// 200 x 4096 764 / 583, 1700 x 1024 179 / 151, 5097 x 832 162 / 141; 8000 x 1024 (252 workgroups and fewer) 203 / 203, 14336 x
// 512 (224) 85 / 88.
template <bool FIRST>
__global__ __launch_bounds__(256, 4) void gptq_trail_small_kernel(const uint16_t* __restrict__ w, float* v, const float* __restrict__ u,
                                                               long N, long K, long base, int n_cols, long col_begin, GqErr err)
{
    __shared__ __attribute__((aligned(16))) float s_a[kGqGroup * kGqGroup], s_b[kGqGroup * kGqGroup];     // errors, rows of U: [c][64]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rg = lane >> 4, cl = lane & 15, wi = wave >> 1, wj = wave & 1;
    const uint32_t n_blocks = (uint32_t)((N + kGqRows - 1) / kGqRows);
    const long cb = blockIdx.x / n_blocks, block = blockIdx.x - (uint32_t)cb * n_blocks;
    const long col0 = col_begin + cb * kGqGroup, row0 = block * kGqRows;
    long eld;
    const float* const eb = gq_err_block(err, block, eld);
    float4 sa[4], sb[4];
    auto fetch = [&](int c0) {
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int c = c0 + (tid >> 4) + 16 * i;
            sa[i] = load_global<float4>(eb + (long)(c >> 2) * eld + (c & 3) * kGqRows + 4 * (tid & 15));
            sb[i] = load_global<float4>(u + (base + c) * K + col0 + 4 * (tid & 15));
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    fetch(0);
    // interleaved: register i of tile (x, y) is row 8 rg + 2 i + x, column 2 cl + y of the wavefront's 32 x 32
    f32x4_t acc[2][2];
    const int r0 = 32 * wi + 8 * rg;
    const long at = col0 + 32 * wj + 2 * cl;
#pragma unroll
    for (int r = 0; r < 8; r++) {
        const long row = min(row0 + r0 + r, N - 1);
        float2 val;
        if constexpr (FIRST) {
            const uint32_t raw = load_global<uint32_t>(w + row * K + at);
            val = make_float2(bf16_lo(raw), bf16_hi(raw));
        } else {
            val = load_global<float2>(v + row * K + at);
        }
        acc[r & 1][0][r >> 1] = val.x;
        acc[r & 1][1][r >> 1] = val.y;
    }
    const float* const ap = s_a + rg * kGqGroup + 32 * wi + 2 * cl;
    const float* const bp = s_b + rg * kGqGroup + 32 * wj + 2 * cl;
#pragma unroll 1
    for (int c0 = 0; c0 < n_cols; c0 += kGqGroup) {
        if (c0 > 0) __syncthreads();                    // the operands before have been read
#pragma unroll
        for (int i = 0; i < 4; i++) {
            *reinterpret_cast<float4*>(s_a + 4 * (tid + 256 * i)) = sa[i];
            *reinterpret_cast<float4*>(s_b + 4 * (tid + 256 * i)) = sb[i];
        }
        __syncthreads();
        fetch(min(c0 + kGqGroup, n_cols - kGqGroup));   // (past the end: the last ones again, unused)
#pragma unroll 4
        for (int kk = 0; kk < kGqGroup / 4; kk++) {
            const float2 av = *reinterpret_cast<const float2*>(ap + kk * 4 * kGqGroup);
            const float2 bv = *reinterpret_cast<const float2*>(bp + kk * 4 * kGqGroup);
            acc[0][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.x, bv.x, acc[0][0], 0, 0, 0);
            acc[0][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.x, bv.y, acc[0][1], 0, 0, 0);
            acc[1][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.y, bv.x, acc[1][0], 0, 0, 0);
            acc[1][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(av.y, bv.y, acc[1][1], 0, 0, 0);
        }
    }
#pragma unroll
    for (int r = 0; r < 8; r++)
        if (row0 + r0 + r < N) store_global(v + (row0 + r0 + r) * K + at, make_float2(acc[r & 1][0][r >> 1], acc[r & 1][1][r >> 1]));
}

// ---------------------------------------------------------------------------
// Hessian of the calibration inputs: hess (+)= X^T X, x [n, K] bf16, fp32 sums on the matrix cores
// (v_mfma_f32_32x32x16_bf16: the products of bf16 numbers are exact in fp32).  Both operands of a tile are
// columns of X, which memory holds row by row: a thread fetches an 8-sample x 8-column block with eight
// 16-byte loads, transposes it in registers and parks eight 16-byte pieces (one column, 8 samples) in LDS,
// chunk position XOR-swizzled by column so that neither the operand reads nor the transposed stores
// collide on banks.  A workgroup owns a 128 x 128 tile on or above the diagonal (64 x 64 per wavefront) and writes the
// mirror image as well.
constexpr int kHsTile = 128;
// Chunk position of column c's 16-byte pieces in LDS: a column is 128 bytes (all 32 banks), so the bank of a
// piece is its chunk position alone.  Eight neighbouring lanes must land on eight positions both when the
// operands are read (lanes = 8 consecutive columns, one chunk) and when the transposed blocks are stored
// (lanes = the same column-in-block of 8 consecutive blocks, one chunk): hence both the low bits and the
// block bits of the column go into the XOR.
__device__ __forceinline__ int hs_swizzle(int c) { return (c ^ (c >> 3)) & 7; }
constexpr int kHsSamples = 64;
constexpr int kHsThreads = 256;

// Bound: per step and workgroup 96 KB through LDS (0.34 us), 1024 cycles of matrix instructions and the transposition beside them; 1.8 us for
// a compute unit's three workgroups.  Three, because K = 4096 has 528 tiles: with two on a compute unit 16 of them were a
// round of their own.  The mirror image leaves 16 bytes a lane at a time.  2048 samples of 4096 columns 102 -> 77 us, 130 samples 38 -> 19.5
// (67 MB written), 2048 of 3072 63 -> 51.
// PARTS: groups of four wavefronts that take the sample steps in turn; their sums meet in LDS, the first part's first.
template <int PARTS>
__global__ __launch_bounds__(PARTS* kHsThreads, PARTS == 1 ? 3 : 2) void gptq_hessian_kernel(const uint16_t* __restrict__ x, long n, long K,
                                                                        int accumulate, float* __restrict__ hess)
{
    __shared__ uint4 s_ops[PARTS][2][kHsTile * (kHsSamples / 8)];      // [part][operand][column][chunk of 8 samples]
    const int part = __builtin_amdgcn_readfirstlane(threadIdx.x / kHsThreads);
    uint4(*const s_op)[kHsTile * (kHsSamples / 8)] = s_ops[part];
    const int tid = threadIdx.x & (kHsThreads - 1);
    const int lane = tid & (kWave - 1), wave = tid / kWave;
    const int ln = lane & 31, kb = lane >> 5;
    // block -> tile (ti, tj), tj >= ti, rows of the upper triangle one after the other
    const int nt = (int)((K + kHsTile - 1) / kHsTile);
    int ti = 0, left = (int)blockIdx.x;
    while (left >= nt - ti) {
        left -= nt - ti;
        ti++;
    }
    const int tj = ti + left;
    const long i0 = (long)ti * kHsTile, j0 = (long)tj * kHsTile;
    // loading role: threads 0..127 the row operand's columns, 128..255 the column operand's
    const int op = tid >> 7;
    const int blk = tid & 127;
    const int sgrp = blk >> 4;                      // which 8 samples of the step's 64
    const int cgrp = blk & 15;                      // which 8 columns of the tile's 128
    const long lcol = (op ? j0 : i0) + 8 * cgrp;
    const int wi = wave >> 1, wj = wave & 1;
    float16_t acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; a++)
#pragma unroll
        for (int b = 0; b < 2; b++)
#pragma unroll
            for (int i = 0; i < 16; i++) acc[a][b][i] = 0.0f;
    uint4 raw[8];
    // Loads without a condition (rows and columns past the end re-read the last ones): behind a test per load the compiler
    // waits for each before the test of the next, and the fetch is no longer in flight during the products.  Columns past
    // the end only reach results that are not stored; rows past the end are cleared below.
    const uint16_t* const xc = x + min(lcol, K - 8);
    auto fetch = [&](long s0) {
#pragma unroll
        for (int r = 0; r < 8; r++) raw[r] = load_global<uint4>(xc + min(s0 + 8 * sgrp + r, n - 1) * K);
        __builtin_amdgcn_sched_barrier(0);
    };
    fetch(part * kHsSamples);
    // (every part makes as many trips; a step past the end adds nothing)
    for (long first = 0; first < n; first += PARTS * kHsSamples) {
        const long s0 = first + part * kHsSamples;
        if (s0 + kHsSamples > n)                    // the last step
#pragma unroll
            for (int r = 0; r < 8; r++)
                if (s0 + 8 * sgrp + r >= n) raw[r] = make_uint4(0u, 0u, 0u, 0u);
        // 8 x 8 transpose of 16-bit values: pair up the rows, split even and odd columns
        uint4 out[8];
#pragma unroll
        for (int dw = 0; dw < 4; dw++) {
            uint32_t even[4], odd[4];
#pragma unroll
            for (int pr = 0; pr < 4; pr++) {
                const uint32_t a = reinterpret_cast<const uint32_t*>(&raw[2 * pr])[dw];
                const uint32_t b = reinterpret_cast<const uint32_t*>(&raw[2 * pr + 1])[dw];
                even[pr] = __builtin_amdgcn_perm(b, a, 0x05040100u);
                odd[pr] = __builtin_amdgcn_perm(b, a, 0x07060302u);
            }
            out[2 * dw] = make_uint4(even[0], even[1], even[2], even[3]);
            out[2 * dw + 1] = make_uint4(odd[0], odd[1], odd[2], odd[3]);
        }
        __syncthreads();                            // the previous step's operand reads are done
#pragma unroll
        for (int i = 0; i < 8; i++) {
            const int c = 8 * cgrp + i;
            s_op[op][c * (kHsSamples / 8) + (sgrp ^ hs_swizzle(c))] = out[i];
        }
        __syncthreads();
        if (first + PARTS * kHsSamples < n) fetch(s0 + PARTS * kHsSamples);          // in flight during the products
#pragma unroll
        for (int ks = 0; ks < kHsSamples / 16; ks++) {
            const int chunk = 2 * ks + kb;
            bf16x8_t fa[2], fb[2];
#pragma unroll
            for (int h = 0; h < 2; h++) {
                const int ca = 64 * wi + 32 * h + ln, cb = 64 * wj + 32 * h + ln;
                fa[h] = __builtin_bit_cast(bf16x8_t, s_op[0][ca * (kHsSamples / 8) + (chunk ^ hs_swizzle(ca))]);
                fb[h] = __builtin_bit_cast(bf16x8_t, s_op[1][cb * (kHsSamples / 8) + (chunk ^ hs_swizzle(cb))]);
            }
#pragma unroll
            for (int a = 0; a < 2; a++)
#pragma unroll
                for (int b = 0; b < 2; b++)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[a], fb[b], acc[a][b], 0, 0, 0);
        }
    }
    if constexpr (PARTS == 2) {
        float* const s_sum = reinterpret_cast<float*>(s_ops);       // [register][thread]
        static_assert(sizeof(s_ops) >= 64 * kHsThreads * sizeof(float), "the second part's sums fit in the operands' place");
        __syncthreads();
        if (part == 1) {
#pragma unroll
            for (int a = 0; a < 4; a++)
#pragma unroll
                for (int i = 0; i < 16; i++) s_sum[(16 * a + i) * kHsThreads + tid] = acc[a >> 1][a & 1][i];
        }
        __syncthreads();
        if (part == 1) return;
#pragma unroll
        for (int a = 0; a < 4; a++)
#pragma unroll
            for (int i = 0; i < 16; i++) acc[a >> 1][a & 1][i] += s_sum[(16 * a + i) * kHsThreads + tid];
    }
    // register i of lane (ln, kb): row 8 (i / 4) + 4 kb + i % 4 of the 32 x 32 tile, column ln: four registers are four neighbours of the
    // mirror image (K and the rows' starts are multiples of 4: all inside or all outside)
#pragma unroll
    for (int a = 0; a < 2; a++)
#pragma unroll
        for (int b = 0; b < 2; b++) {
            const long c = j0 + 64 * wj + 32 * b + ln;
            if (c >= K) continue;
#pragma unroll
            for (int i0r = 0; i0r < 4; i0r++) {
                const long r = i0 + 64 * wi + 32 * a + 8 * i0r + 4 * kb;
                if (r >= K) continue;
                float val[4];
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    val[i] = acc[a][b][4 * i0r + i];
                    if (accumulate) val[i] += hess[(r + i) * K + c];
                    hess[(r + i) * K + c] = val[i];
                }
                if (ti != tj) store_global(hess + c * K + r, make_float4(val[0], val[1], val[2], val[3]));
            }
        }
}

// ---------------------------------------------------------------------------
// Factor of the inverse Hessian: U upper triangular, (H + damping)^-1 = U^T U.
// With J the order-reversing permutation and A = J (H + damping) J = L L^T (plain Cholesky), U = J L^-1 J.
// Cholesky and inverse run together, block of 64 columns after block: L^-1 is what forward substitution makes of the
// unit vectors, and the columns of A to the left of a block are dead by the time their part of the substitution starts,
// so both live in one lower triangle v.  Step k makes P, the block row that every later row is corrected with, 64 x K: for rows
// j below the block the new column block of L (P[c, j] = L[j, 64 k + c]: row j of A solved against L_kk), for columns j left of
// it the finished rows of L^-1 (column j of the right-hand sides solved against L_kk), the inverse of L_kk itself in between
// (unit vectors); the finished rows go to their mirrored place in u.  What P does to the rest:
//   v[i, j] -= sum_c P[c, i] P[c, j] for the rows i below the block, columns j <= i (columns of the block itself start from zero)

// damping = damp * mean of the diagonal, a zero diagonal entry counting as (and becoming) 1
__global__ __launch_bounds__(256) void gptq_damping_kernel(const float* __restrict__ hess, long K, float damp,
                                                           float* __restrict__ lambda)
{
    __shared__ double s_part[256];
    double acc = 0.0;
    // (eight entries requested together, added in order: one by one, K = 4096 took 16 trips to memory: 7.4 -> 5.7 us)
    for (long i0 = threadIdx.x; i0 < K; i0 += 8 * 256) {
        float dg[8];
#pragma unroll
        for (int e = 0; e < 8; e++) {
            const long i = min(i0 + 256 * e, K - 1);
            dg[e] = load_global<float>(hess + i * K + i);
        }
#pragma unroll
        for (int e = 0; e < 8; e++)
            if (i0 + 256 * e < K) acc += (dg[e] == 0.0f) ? 1.0 : (double)dg[e];
    }
    s_part[threadIdx.x] = acc;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) s_part[threadIdx.x] += s_part[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) *lambda = (float)((double)damp * s_part[0] / (double)K);
}

// v = the lower triangle of J (H + damping) J, whole 64 x 64 blocks, a workgroup per 16 rows x 256 columns, its loads
// all in flight at once (64 x 256 left half of the chip without work: 18 -> 13 us at K = 4096)
constexpr int kGqReverseRows = 16;
__global__ __launch_bounds__(256) void gptq_reverse_kernel(const float* __restrict__ hess, long K,
                                                           const float* __restrict__ lambda, float* __restrict__ v)
{
    const long row0 = (long)blockIdx.y * kGqReverseRows;
    const long j = (long)blockIdx.x * 256 + threadIdx.x;
    if (j >= (row0 / kGqGroup + 1) * kGqGroup) return;
    const float add = *lambda;
    float val[kGqReverseRows];
#pragma unroll
    for (int r = 0; r < kGqReverseRows; r++) val[r] = load_global<float>(hess + (K - 1 - row0 - r) * K + (K - 1 - j));
#pragma unroll
    for (int r = 0; r < kGqReverseRows; r++) {
        if (row0 + r == j) val[r] = ((val[r] == 0.0f) ? 1.0f : val[r]) + add;
        v[(row0 + r) * K + j] = val[r];
    }
}

// The 16 columns p .. p + 15 of the Cholesky factor of the 64 x 64 block in LDS (row stride 68), by one wavefront: a lane per
// row with its 16 values in registers, pivots and multipliers through v_readlane.  Also the 16 x 16 block on the diagonal as
// the solving wavefronts read it (s_q[c][row % 4][row / 4]) and the diagonal with its reciprocals.
constexpr int kGqLd = kGqGroup + 4;
__device__ __forceinline__ void gq_chol_piece(float* s_m, int p, float* s_q, float2* s_inv)
{
    const int row = threadIdx.x & (kWave - 1);
    float a[16], dg = 0.0f;
    bool ordinary = true;
#pragma unroll
    for (int c = 0; c < 4; c++) {
        const float4 t = *reinterpret_cast<const float4*>(s_m + row * kGqLd + p + 4 * c);
        a[4 * c] = t.x; a[4 * c + 1] = t.y; a[4 * c + 2] = t.z; a[4 * c + 3] = t.w;
    }
#pragma unroll
    for (int c = 0; c < 16; c++) {
        const float d = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(a[c]), p + c));
        // square root and quotient: the hardware's estimate of 1 / sqrt(d) and one residual step each (finite operands; see
        // the step kernel for infinite ones)
        const float y = __builtin_amdgcn_rsqf(d);
        const float s0 = d * y, l0 = a[c] * y;
        const float sq = __builtin_fmaf(__builtin_fmaf(-s0, s0, d), 0.5f * y, s0);
        float l = __builtin_fmaf(__builtin_fmaf(-sq, l0, a[c]), y, l0);
        l = (row == p + c) ? sq : l;
        ordinary &= d > 1e-30f && d < 1e30f;
        a[c] = l;
#pragma unroll
        for (int j = c + 1; j < 16; j++) {
            const float lj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(l), p + j));
            a[j] = __builtin_fmaf(-l, lj, a[j]);
        }
    }
    if (!ordinary) {                                                // the same in every lane
        // a pivot so large or small that the estimate's steps may leave the range (or none at all: NaN): root and division as
        // they are, in LDS
#pragma unroll 1
        for (int c = 0; c < 16; c++) {
            const float root = sqrtf(s_m[(p + c) * kGqLd + p + c]);
            const float l = (row == p + c) ? root : s_m[row * kGqLd + p + c] / root;
            s_m[row * kGqLd + p + c] = l;
            for (int j = c + 1; j < 16; j++)
                s_m[row * kGqLd + p + j] = __builtin_fmaf(-l, s_m[(p + j) * kGqLd + p + c], s_m[row * kGqLd + p + j]);
        }
#pragma unroll
        for (int c = 0; c < 16; c++) a[c] = s_m[row * kGqLd + p + c];
    }
#pragma unroll
    for (int c = 0; c < 4; c++)
        *reinterpret_cast<float4*>(s_m + row * kGqLd + p + 4 * c) = make_float4(a[4 * c], a[4 * c + 1], a[4 * c + 2], a[4 * c + 3]);
    const int lr = row - p;
    if (lr >= 0 && lr < 16) {
#pragma unroll
        for (int c = 0; c < 16; c++) {
            s_q[(p + c) * kGqChunk + (lr & 3) * 4 + (lr >> 2)] = a[c];
            dg = (lr == c) ? a[c] : dg;
        }
        s_inv[row] = make_float2(dg, 1.0f / dg);
    }
}

// One 16 x 16 tile (t, tt) of the block loses the products of the 16 columns from p on: m[row, col] = fma(-L[row, c], L[col, c],
// m[row, col]), c ascending.
__device__ __forceinline__ void gq_chol_tile(float* s_m, int p, int t, int tt)
{
    const int lane = threadIdx.x & (kWave - 1), rg = lane >> 4, cl = lane & 15;
    float* const at = s_m + (16 * t + 4 * rg) * kGqLd + 16 * tt + cl;
    f32x4_t acc;
    float x[4], y[4];
#pragma unroll
    for (int i = 0; i < 4; i++) acc[i] = at[i * kGqLd];
#pragma unroll
    for (int kk = 0; kk < 4; kk++) {
        x[kk] = -s_m[(16 * t + cl) * kGqLd + p + 4 * kk + rg];
        y[kk] = s_m[(16 * tt + cl) * kGqLd + p + 4 * kk + rg];
    }
#pragma unroll
    for (int kk = 0; kk < 4; kk++) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[kk], y[kk], acc, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; i++) at[i * kGqLd] = acc[i];
}

// Where P of step s has its 64 columns `block`: in v's block row s, which nothing else needs any more (to the left of the
// diagonal in the place of the rows it was solved from, to the right in the unused upper triangle), its own diagonal block, which
// every workgroup of the step reads, in slot s.
__device__ __forceinline__ const float* gq_p_block(const float* v, long K, const float* slots, long s, long block, long& ld)
{
    ld = (block == s) ? kGqGroup : K;
    return (block == s) ? slots + s * kGqGroup * kGqGroup : v + s * kGqGroup * K + block * kGqGroup;
}

// Step k of the factorisation in one launch.  The first K / 64 workgroups solve: workgroup jb takes step k - 1 out of the diagonal
// block and out of its own block of v, makes the diagonal block's Cholesky factor and, 16 columns behind it, the substitution.
// The others bring the rest of v forward, steps in pairs (a panel: steps 2 q and 2 q + 1), so that a block of v is read and
// written once per panel:
//   k = 2 q + 2   panel q into the block pairs q + 1 and q + 2 (columns and rows) and into some of the blocks behind them
//   k = 2 q + 3   panel q into the other blocks; step 2 q + 2 alone into block row and column 2 q + 4, which step 2 q + 4 needs
// The launch lasts as long as its chain, or, for the first steps of a large K, as the matrix products: 1 us to start, 2 for the
// operands, 2 of products, 5 stages of 1.4 to 1.9 in which one wavefront factors 16 columns, three bring the diagonal block
// forward and four substitute the 16 columns before.  K = 4096: 20 us a step on average, 15 to 17 for the last ones; as two launches a step (substitution
// 9 us, update and Cholesky 13 to 25 with v crossing memory in every one of them) 28.
// The quotient is the product with the reciprocal and one residual step.  For finite operands that differs from a division
// in the last place at most; an infinite operand or quotient gives NaN where the division gives infinity, but it has no
// place in a positive definite matrix: what it is subtracted from, a later pivot, becomes NaN either way.
constexpr int kGqStepThreads = 512;
constexpr int kGqStepLds = 3 * kGqGroup * kGqGroup;                 // floats: a tile's operands of 64 columns c

// Tiles (pairs of block rows x pairs of block columns) of panel q: `near` of the pairs q + 1 and q + 2 and `first` of the
// others in the first launch, `later` in the second.  single: half tiles that the second launch brings forward by one step.
struct GqWide {
    long q, pairs, near, first, later, single;
};
static inline GqWide gq_wide(long nb, long k)
{
    GqWide w;
    w.q = k / 2 - 1;
    w.pairs = (nb + 1) / 2;
    w.near = w.first = w.later = w.single = 0;
    if (k + 1 >= nb) return w;                                      // the last step leaves nothing behind
    if (w.q >= 0) {
        w.near = w.pairs + (w.q + 2 < w.pairs ? w.pairs - 1 : 0);
        // the others: pairs si >= q + 3, and si - 1 of the si + 1 column pairs each
        long rest = ((w.pairs - 1) * (w.pairs - 2) - (w.q + 2) * (w.q + 1)) / 2;
        if (rest < 0) rest = 0;
        w.first = (w.near + rest) / 2 - w.near;
        if (w.first < 0) w.first = 0;
        w.later = rest - w.first;
    }
    if (k & 1) w.single = nb - (k + 1) + w.q + 2;                   // block column k + 1 from the diagonal down, block row k + 1
    return w;
}
static inline long gq_wide_blocks(const GqWide& w, long k) { return (k & 1) ? w.single + 2 * w.later : 2 * (w.near + w.first); }

__global__ __launch_bounds__(kGqStepThreads, 6) void gptq_step_kernel(float* v, long K, long k, float* slots, float* __restrict__ u,
                                                                     GqWide wide)
{
    extern __shared__ __attribute__((aligned(16))) float s_all[];   // kGqStepLds at least
    const long nb = K / kGqGroup;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rg = lane >> 4, cl = lane & 15;
    if ((long)blockIdx.x >= nb) {
        // ---- 64 x 128, a block row of a tile, 32 x 32 of it a wavefront
        const long last = nb - 1, q = wide.q;
        const int wi = wave >> 2, wq = wave & 3;
        const long at0 = (long)blockIdx.x - nb, n_single = (k & 1) ? wide.single : 0;
        const bool single = at0 < n_single;
        long ib, sj;
        if (single) {
            const long below = nb - (k + 1);
            ib = at0 < below ? k + 1 + at0 : k + 1;
            sj = at0 < below ? q + 2 : at0 - below;
        } else {
            const long half = at0 - n_single, tile = half >> 1, below = wide.pairs - q - 1;
            long si;
            if (!(k & 1) && tile < wide.near) {
                if (tile < below) { si = q + 1 + tile; sj = q + 1; }
                else if (tile < wide.pairs) { si = q + 1; sj = tile - below; }
                else if (tile < wide.pairs + below - 1) { si = q + 2 + tile - wide.pairs; sj = q + 2; }
                else { si = q + 2; sj = tile - wide.pairs - (below - 1); }
            } else {
                // m = si - 1 column pairs (without q + 1 and q + 2) of every pair si >= q + 3
                const long r = ((k & 1) ? tile + wide.first : tile - wide.near) + (q + 2) * (q + 1) / 2;
                long m = (long)((sqrt(8.0 * (double)r + 1.0) + 1.0) * 0.5);
                while (m * (m - 1) / 2 > r) m--;
                while ((m + 1) * m / 2 <= r) m++;
                si = m + 1;
                sj = r - m * (m - 1) / 2;
                if (sj >= q + 1) sj += 2;
            }
            ib = 2 * si + (half & 1);
        }
        const long s0 = single ? k - 1 : 2 * q;
        const long jb = min(2 * sj + (wq >> 1), last);
        if (ib > last || (!single && ib == s0 + 2)) return;         // (the same in the whole workgroup)
        const bool mine = 2 * sj + (wq >> 1) <= last && jb <= ib && (single ? jb == k + 1 || (ib == k + 1 && jb != k) : jb != s0 + 2);
        // the panel's two steps one after the other through LDS, 64 columns c at a time: rows [c][64], columns [c][128]; the
        // second step's operands are on their way while the first one's are multiplied
        float4 sa[2], sb[4];
        auto fetch = [&](long s) {
            long ld;
            const float* const pa = gq_p_block(v, K, slots, s, ib, ld);
#pragma unroll
            for (int i = 0; i < 2; i++) sa[i] = load_global<float4>(pa + ((tid >> 4) + 32 * i) * ld + 4 * (tid & 15));
            const int f4 = tid & 31;
            const float* const pb = gq_p_block(v, K, slots, s, min(2 * sj + (f4 >> 4), last), ld);
#pragma unroll
            for (int i = 0; i < 4; i++) sb[i] = load_global<float4>(pb + ((tid >> 5) + 16 * i) * ld + 4 * (f4 & 15));
            __builtin_amdgcn_sched_barrier(0);
        };
        float* const s_b = s_all + kGqGroup * kGqGroup;
        auto park = [&] {
#pragma unroll
            for (int i = 0; i < 2; i++) *reinterpret_cast<float4*>(s_all + 4 * (tid + kGqStepThreads * i)) = sa[i];
#pragma unroll
            for (int i = 0; i < 4; i++) *reinterpret_cast<float4*>(s_b + 4 * (tid + kGqStepThreads * i)) = sb[i];
            __syncthreads();
        };
        // interleaved as in GqTile, with two row and two column tiles: register i of tile (x, y) is row 8 rg + 2 i + x, column
        // 2 cl + y
        f32x4_t acc[2][2];
        auto multiply = [&] {
            const float* ap = s_all + rg * kGqGroup + 32 * wi + 2 * cl;
            const float* bp = s_b + rg * 128 + 32 * wq + 2 * cl;
#pragma unroll 4
            for (int kk = 0; kk < kGqGroup / 4; kk++) {
                const float2 av = *reinterpret_cast<const float2*>(ap + kk * 4 * kGqGroup);
                const float2 bv = *reinterpret_cast<const float2*>(bp + kk * 512);
                acc[0][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(-av.x, bv.x, acc[0][0], 0, 0, 0);
                acc[0][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(-av.x, bv.y, acc[0][1], 0, 0, 0);
                acc[1][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(-av.y, bv.x, acc[1][0], 0, 0, 0);
                acc[1][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(-av.y, bv.y, acc[1][1], 0, 0, 0);
            }
        };
        fetch(s0);
        const uint32_t off = 8 * rg * (uint32_t)K + 2 * cl;
        float* const dst = v + (ib * kGqGroup + 32 * wi) * K + jb * kGqGroup + 32 * (wq & 1);
#pragma unroll
        for (int r = 0; r < 8; r++) {
            float2 val = make_float2(0.0f, 0.0f);       // (block columns of the panel itself: L^-1's part starts here)
            if (jb != s0 && (single || jb != s0 + 1)) val = load_global<float2>(dst + r * K + off);
            acc[r & 1][0][r >> 1] = val.x;
            acc[r & 1][1][r >> 1] = val.y;
        }
        park();
        if (!single) fetch(s0 + 1);
        multiply();
        if (!single) {
            __syncthreads();                            // the first step's operands have been read
            park();
            if (jb == s0 + 1) {                         // ... with the panel's second step
#pragma unroll
                for (int x = 0; x < 2; x++) acc[x][0] = acc[x][1] = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
            }
            multiply();
        }
        if (!mine) return;
#pragma unroll
        for (int r = 0; r < 8; r++) store_global(dst + r * K + off, make_float2(acc[r & 1][0][r >> 1], acc[r & 1][1][r >> 1]));
        return;
    }
    // ---- solve
    float* const s_m = s_all;                                       // diagonal block, 64 rows of 68
    float* const s_x = s_m + kGqGroup * kGqLd;                      // own block, [column j][c], 64 rows of 68
    float* const s_q = s_x + kGqGroup * kGqLd;                      // 16 x 16 blocks of the factor's diagonal
    float2* const s_inv = reinterpret_cast<float2*>(s_q + kGqGroup * kGqChunk);
    float* const s_e = reinterpret_cast<float*>(s_inv + kGqGroup);  // [wavefront][c of the 16][column], negated
    static_assert(2 * kGqGroup * kGqLd + kGqGroup * kGqChunk + 2 * kGqGroup + kGqChunk * kGqGroup <= kGqStepLds, "the solver's blocks fit");
    __builtin_amdgcn_s_setprio(3);                                  // the launch's longest chain, beside wavefronts that only add work
    const long jb = blockIdx.x, base = k * kGqGroup;
    {
        // columns of block k and of the own block of step k - 1's P into LDS, [block k, own][c][column]: all requested at once (the
        // workgroups of the launch before left them in other L2s, a microsecond away)
        const long before = k - 1;
        const bool with_own = jb > k || (jb < k && k > 0);
        float4 stage[2][2];
#pragma unroll
        for (int b = 0; b < 2; b++)
            if (k > 0 && (b == 0 || with_own)) {
                long ld;
                const float* const from = gq_p_block(v, K, slots, before, b ? jb : k, ld) + (tid >> 4) * ld + 4 * (tid & 15);
#pragma unroll
                for (int i = 0; i < 2; i++) stage[b][i] = load_global<float4>(from + 32 * i * ld);
            }
        // wavefronts 0..3: a quadrant each of the diagonal block; 4..7: of the own one (below the diagonal transposed: rows j)
        const bool own = wave >= 4;
        const int w4 = wave & 3, wi = w4 >> 1, wj = w4 & 1, ln = lane & 31, h = lane >> 5;
        const long rows = own && jb > k ? jb : k, cols = own && jb < k ? jb : k;
        float16_t acc;
        const float* const src = v + (rows * kGqGroup + 32 * wi + 4 * h) * K + cols * kGqGroup + 32 * wj + ln;
#pragma unroll
        for (int i = 0; i < 16; i++) {
            acc[i] = 0.0f;                                          // (block column k - 1: L^-1's part starts with its own step)
            if (own && jb == k) acc[i] = (32 * wi + 8 * (i >> 2) + 4 * h + (i & 3) == 32 * wj + ln) ? 1.0f : 0.0f;
            else if (cols != before) acc[i] = src[(long)(8 * (i >> 2) + (i & 3)) * K];
        }
        __builtin_amdgcn_sched_barrier(0);
        if (k > 0) {
#pragma unroll
            for (int b = 0; b < 2; b++)
#pragma unroll
                for (int i = 0; i < 2; i++)
                    *reinterpret_cast<float4*>(s_all + b * kGqGroup * kGqGroup + 4 * (tid + kGqStepThreads * i)) = stage[b][i];
        }
        __syncthreads();
        if (k > 0 && !(own && jb == k) && wave != 1) {              // (wavefront 1: above the diagonal, not needed)
            const float* const ap = s_all + (rows == k ? 0 : kGqGroup * kGqGroup) + h * kGqGroup + 32 * wi + ln;
            const float* const bp = s_all + (cols == k ? 0 : kGqGroup * kGqGroup) + h * kGqGroup + 32 * wj + ln;
#pragma unroll 8
            for (int c = 0; c < kGqGroup; c += 2) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(-ap[c * kGqGroup], bp[c * kGqGroup], acc, 0, 0, 0);
        }
        __syncthreads();                                            // the operands have been read
#pragma unroll
        for (int i = 0; i < 16; i++) {
            const int r = 32 * wi + 8 * (i >> 2) + 4 * h + (i & 3), c = 32 * wj + ln;
            if (!own) s_m[r * kGqLd + c] = acc[i];
            else if (jb > k) s_x[r * kGqLd + c] = acc[i];
            else s_x[c * kGqLd + r] = acc[i];
        }
    }
    __syncthreads();
    const int w4 = wave & 3, rr = lane >> 2, q = lane & 3;
    const long j = jb * kGqGroup + 16 * w4 + rr;                    // substitution: four lanes per column
    float* const xr = s_x + 16 * w4 * kGqLd;
    float* const se = s_e + w4 * kGqChunk * 16;
    float* const pj = jb == k ? slots + k * kGqGroup * kGqGroup + q * kGqGroup + 16 * w4 + rr : v + (base + q) * K + j;
    const long pld = jb == k ? kGqGroup : K;
    float* const uj = u + (K - 1 - base - q) * K + (K - 1 - j);
#pragma unroll 1
    for (int s = 0; s < 5; s++) {
        // the 16 columns before into the present ones, a tile a wavefront
        if (s > 0 && s + wave < 4) gq_chol_tile(s_m, 16 * s - 16, s + wave, s);
        __syncthreads();
        if (wave == 0) {
            if (s < 4) gq_chol_piece(s_m, 16 * s, s_q, s_inv);
        } else if (wave < 4) {
            // ... and into what is behind them: tiles (2, 2), (3, 2), (3, 3), then (3, 3)
            if (s == 1) gq_chol_tile(s_m, 0, wave == 1 ? 2 : 3, wave == 3 ? 3 : 2);
            else if (s == 2 && wave == 1) gq_chol_tile(s_m, 16, 3, 3);
        } else if (s > 0) {
            const int t0 = 16 * (s - 1);
            float x[4], keep = 0.0f;
#pragma unroll
            for (int i = 0; i < 4; i++) x[i] = xr[rr * kGqLd + t0 + 4 * i + q];
            const float4* const sd = reinterpret_cast<const float4*>(s_q + t0 * kGqChunk + 4 * q);
#pragma unroll
            for (int i = 0; i < kGqChunk; i++) {
                const int k4 = i / 4, c = i % 4;
                const float xi = c == 0 ? quad_bcast<0>(x[k4]) : c == 1 ? quad_bcast<1>(x[k4]) : c == 2 ? quad_bcast<2>(x[k4]) : quad_bcast<3>(x[k4]);
                const float2 dg = s_inv[t0 + i];
                const float e0 = xi * dg.y;
                const float e = __builtin_fmaf(__builtin_fmaf(-dg.x, e0, xi), dg.y, e0);    // the quotient: one residual step
                keep = (q == c) ? e : keep;
                if (c == 3) {
                    pj[(long)(t0 + 4 * k4) * pld] = keep;
                    uj[-(long)(t0 + 4 * k4) * K] = (jb > k) ? 0.0f : keep;
                    se[(4 * k4 + q) * 16 + rr] = -keep;
                }
                const float4 d4 = sd[i * (kGqChunk / 4)];
                const float dd[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
                for (int m = (c == 3) ? k4 + 1 : k4; m < 4; m++) x[m] = __builtin_fmaf(-e, dd[m], x[m]);
            }
            // ... and onto the columns behind them
            float a[4];
#pragma unroll
            for (int kk = 0; kk < 4; kk++) a[kk] = se[4 * kk * 16 + lane];
            for (int tt = s; tt < 4; tt++) {
                float* const at = xr + 4 * rg * kGqLd + 16 * tt + cl;
                f32x4_t acc;
                float y[4];
#pragma unroll
                for (int i = 0; i < 4; i++) acc[i] = at[i * kGqLd];
#pragma unroll
                for (int kk = 0; kk < 4; kk++) y[kk] = s_m[(16 * tt + cl) * kGqLd + t0 + 4 * kk + rg];
#pragma unroll
                for (int kk = 0; kk < 4; kk++) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[kk], y[kk], acc, 0, 0, 0);
#pragma unroll
                for (int i = 0; i < 4; i++) at[i * kGqLd] = acc[i];
            }
        }
        __syncthreads();
    }
}

}  // namespace dymoe

extern "C" {

size_t dymoe_gptq_workspace_bytes(long N, long K)
{
    if (N <= 0 || K <= 0) return 0;
    return dymoe::gq_round256((size_t)N * (size_t)K * 4) + dymoe::gq_tail_bytes(N);
}

int dymoe_gptq_quantize_pack(dymoe_ctx* ctx, const void* w_bf16, const float* u, long N, long K, int bits, int group,
                             uint8_t* codes, void* scale, void* zero, void* workspace, size_t workspace_bytes,
                             void* stream)
{
    using namespace dymoe;
    DYMOE_REQUIRE(w_bf16 && u && codes && scale && zero && workspace);
    DYMOE_REQUIRE(N > 0 && K > 0 && (bits == 2 || bits == 4 || bits == 8));
    DYMOE_REQUIRE(group == kGqGroup && K % kGqGroup == 0);
    DYMOE_REQUIRE(N * K < ((long)1 << 40));
    DYMOE_REQUIRE(dymoe_aligned(w_bf16, 16) && dymoe_aligned(u, 16) && dymoe_aligned(codes, 16) &&
                  dymoe_aligned(scale, 2) && dymoe_aligned(zero, 2) && dymoe_aligned(workspace, 256));
    if (workspace_bytes < dymoe_gptq_workspace_bytes(N, K)) return DYMOE_ENOSPC;
    if (!ctx) return DYMOE_ENOCTX;
    hipStream_t st = (hipStream_t)stream;
    const long n_blocks = gq_row_blocks(N);
    float* v = reinterpret_cast<float*>(workspace);
    float* tail = reinterpret_cast<float*>((char*)workspace + gq_round256((size_t)N * (size_t)K * 4));
    const int panel = gq_panel(N);
    const uint16_t* w = (const uint16_t*)w_bf16;
    uint16_t* sc = (uint16_t*)scale;
    uint16_t* zr = (uint16_t*)zero;
    for (long base = 0; base < K; base += panel * kGqGroup) {
        const long left = (K - base) / kGqGroup;
        const int groups = (int)(left < panel ? left : panel);
        const long next = base + groups * kGqGroup;
        const GqErr err = {v + base, K, tail, N / kGqRows};
        auto go = [&](auto kernel) {
            dymoe_launch(ctx, DYMOE_K_GPTQ_GROUP, kernel, dim3((unsigned)n_blocks), dim3(256), 0, st, w, v, u, N, K, base,
                         groups, err, codes, sc, zr);
        };
        const bool first = base == 0;
        if (bits == 8) first ? go(gptq_group_kernel<8, true>) : go(gptq_group_kernel<8, false>);
        else if (bits == 4) first ? go(gptq_group_kernel<4, true>) : go(gptq_group_kernel<4, false>);
        else first ? go(gptq_group_kernel<2, true>) : go(gptq_group_kernel<2, false>);
        DYMOE_HIP_LAUNCH_CHECK();
        if (next >= K) break;
        const long row_pairs = (n_blocks + 1) / 2, col_pairs = (K - next + 2 * kGqGroup - 1) / (2 * kGqGroup);
        auto trail = [&](auto kernel, long blocks) {
            dymoe_launch(ctx, DYMOE_K_GPTQ_TRAIL, kernel, dim3((unsigned)blocks), dim3(256), 0, st, w, v, u, N, K, base, groups * kGqGroup,
                         next, err);
        };
        if (4 * row_pairs * col_pairs <= 3L * ctx->num_cu) {
            const long blocks = n_blocks * ((K - next) / kGqGroup);
            first ? trail(gptq_trail_small_kernel<true>, blocks) : trail(gptq_trail_small_kernel<false>, blocks);
        } else {
            const long blocks = 8 * ((row_pairs + 7) / 8) * col_pairs;
            first ? trail(gptq_trail_kernel<true>, blocks) : trail(gptq_trail_kernel<false>, blocks);
        }
        DYMOE_HIP_LAUNCH_CHECK();
    }
    return DYMOE_OK;
}

int dymoe_gptq_hessian(dymoe_ctx* ctx, const void* x_bf16, long n, long K, int accumulate, float* hess, void* stream)
{
    using namespace dymoe;
    DYMOE_REQUIRE(x_bf16 && hess && n > 0 && K > 0 && K % 8 == 0 && (accumulate == 0 || accumulate == 1));
    DYMOE_REQUIRE(K <= 65536 && dymoe_aligned(x_bf16, 16) && dymoe_aligned(hess, 16));
    if (!ctx) return DYMOE_ENOCTX;
    const long nt = (K + kHsTile - 1) / kHsTile;
    const long tiles = nt * (nt + 1) / 2;
    auto go = [&](auto kernel, int parts) {
        dymoe_launch(ctx, DYMOE_K_GPTQ_HESSIAN, kernel, dim3((unsigned)tiles), dim3((unsigned)(parts * kHsThreads)), 0, (hipStream_t)stream,
                     (const uint16_t*)x_bf16, n, K, accumulate, hess);
    };
    // Not more tiles than compute units: a tile's steps are a chain of 1.3 us each (load, transpose, store, barriers,
    // products), and two parts of a workgroup share it.  One part / two, us: 4096 samples of 256 columns 65.7 / 50.8, 2216 of
    // 960 39.9 / 32.1, 2048 of 2048 38.9 / 32.0, 2048 of 2816 43.0 / 38.4, 1000 of 512 20.2 / 17.0; 300 of 960 10.1 / 10.4 (the
    // exchange costs more than three steps less give).  With more tiles the other workgroups of a compute unit fill the gaps: 2048 of
    // 3072 50.3 / 60.3, of 4096 77.6 / 91.8.
    if (tiles <= ctx->num_cu && n > 8 * kHsSamples) go(gptq_hessian_kernel<2>, 2);
    else go(gptq_hessian_kernel<1>, 1);
    DYMOE_HIP_LAUNCH_CHECK();
    return DYMOE_OK;
}

size_t dymoe_gptq_factor_workspace_bytes(long K)
{
    if (K <= 0) return 0;
    // the triangle that becomes factor and inverse, a 64 x 64 block per step, the damping (in an area of 64 x 64 + 1)
    return dymoe::gq_round256((size_t)K * (size_t)K * 4) + dymoe::gq_round256((size_t)dymoe::kGqGroup * (size_t)K * 4) +
           dymoe::gq_round256(((size_t)dymoe::kGqGroup * dymoe::kGqGroup + 1) * 4);
}

int dymoe_gptq_factor(dymoe_ctx* ctx, const float* hess, long K, float damp, float* u, void* workspace,
                      size_t workspace_bytes, void* stream)
{
    using namespace dymoe;
    DYMOE_REQUIRE(hess && u && workspace && K > 0 && K % kGqGroup == 0 && K <= 65536 && damp >= 0.0f);
    DYMOE_REQUIRE(dymoe_aligned(hess, 16) && dymoe_aligned(u, 16) && dymoe_aligned(workspace, 256));
    DYMOE_REQUIRE((const void*)hess != (const void*)u);
    if (workspace_bytes < dymoe_gptq_factor_workspace_bytes(K)) return DYMOE_ENOSPC;
    if (!ctx) return DYMOE_ENOCTX;
    hipStream_t st = (hipStream_t)stream;
    const size_t mat = gq_round256((size_t)K * (size_t)K * 4);
    float* v = reinterpret_cast<float*>(workspace);
    float* slots = reinterpret_cast<float*>((char*)workspace + mat);                    // 64 x 64 per step
    float* lambda = reinterpret_cast<float*>((char*)slots + gq_round256((size_t)kGqGroup * (size_t)K * 4));
    hipLaunchKernelGGL(gptq_damping_kernel, dim3(1), dim3(256), 0, st, hess, K, damp, lambda);
    hipLaunchKernelGGL(gptq_reverse_kernel, dim3((unsigned)((K + 255) / 256), (unsigned)(K / kGqReverseRows)), dim3(256), 0, st, hess, K,
                       (const float*)lambda, v);
    DYMOE_HIP_LAUNCH_CHECK();
    const long nb = K / kGqGroup;
    for (long k = 0; k < nb; k++) {
        const GqWide wide = gq_wide(nb, k);
        const long blocks = nb + gq_wide_blocks(wide, k);
        // Three workgroups fit on a compute unit, but while all of a launch's are resident together that puts two tiles beside a
        // solver and three elsewhere, and the launch waits for the solver: 64 KB of LDS let two in, and the last tiles go
        // where one has ended (K = 4096: 1.41 -> 1.35 ms).  Beyond one filling the tiles are what it waits for (14336: 28.4
        // with two, 25.4 with three).
        const size_t lds = blocks <= 3L * ctx->num_cu ? 4 * kGqGroup * kGqGroup * 4 : kGqStepLds * 4;
        dymoe_launch(ctx, DYMOE_K_GPTQ_FACTOR, gptq_step_kernel, dim3((unsigned)blocks), dim3(kGqStepThreads), lds, st, v, K, k, slots, u,
                     wide);
        DYMOE_HIP_LAUNCH_CHECK();
    }
    return DYMOE_OK;
}

}  // extern "C"
