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
// Rows are independent, columns are not.  Columns go in panels of 256 (four groups of 64), a launch each, which does two things side by side:
//   the panel      32 rows a workgroup: their values lose the errors of the panel before, then group after group is quantised
//                  column by column (a chain of dependent steps: four lanes share a row, a lane every fourth column) and its errors
//                  corrected in the panel's later groups; codes, scale, zero and the errors e are written;
//   the rest       v[:, j] for the columns behind the panel loses the errors of the panel before: 256 chained fmas per element.
// The working copy v of the matrix (fp32) lives in the caller's workspace.
#include <type_traits>

#include "common.hpp"
#include "gptq_steps.hpp"

namespace dymoe {

constexpr int kGqGroup = 64;        // columns per group
constexpr int kGqRows = 32;         // rows per row block
constexpr int kGqPanel = 4;         // groups per panel
constexpr int kGqChunk = 16;        // columns per piece of a group's chain

typedef float f32x4_t __attribute__((ext_vector_type(4)));

static inline size_t gq_round256(size_t v) { return (v + 255) & ~(size_t)255; }
static inline long gq_row_blocks(long N) { return (N + kGqRows - 1) / kGqRows; }

// Groups per panel.  Below 64 rows half a panel, so that the errors of two panels of a ragged block find room in the buffer.
static inline int gq_panel(long N) { return (N < 2 * kGqRows) ? kGqPanel / 2 : kGqPanel; }

// bytes of the ragged row block's errors, two panels' columns of 32 rows; no ragged block, no buffer (the buffer also where the last 32 of 64 rows are missing)
static inline size_t gq_tail_bytes(long N)
{
    return (N % (2 * kGqRows)) ? 2 * (size_t)gq_panel(N) * kGqGroup * kGqRows * sizeof(float) : 0;
}

// Where the (negated) errors of a panel of `cols` columns are kept until the next launch has used them.  The panel's own columns of
// v are dead once its values are in registers, and a row block's 32 x cols of them hold its cols x 32 errors exactly:
// element (column c of the panel, row r of the block) sits in row c / (cols / 32) of the block at offset (c % (cols / 32)) * 32 + r.  The
// ragged last row block has too few rows for that and uses a linear buffer of the same arrangement (row stride cols).
struct GqErr {
    float* whole;     // v + first column of the panel
    float* tail;      // linear buffer of the ragged block
    long ld;          // row stride of v
    long full_blocks;
    int cols;
};
__device__ __forceinline__ float* gq_err_block(const GqErr& g, long block, long& ld)
{
    const bool full = block < g.full_blocks;
    ld = full ? g.ld : g.cols;
    return full ? g.whole + block * kGqRows * g.ld : g.tail;
}
// of element (c, r) within a block
__device__ __forceinline__ long gq_err_at(const GqErr& g, long ld, int c, int r)
{
    const int shift = (g.cols == kGqPanel * kGqGroup) ? 3 : 2;                          // 8 or 4 columns c a row
    return (long)(c >> shift) * ld + (c & ((1 << shift) - 1)) * kGqRows + r;
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

// LDS of a panel's workgroup, floats: first two buffers for the corrections of the panel before (16 columns c: 256 columns of U and 32 rows
// of errors), then the corrected values, then the errors [column][row]; behind them what is there throughout.
constexpr int kGqULd = kGqPanel * kGqGroup + 16;                    // row stride of U in a buffer: c and c + 1 on other banks
constexpr int kGqStage = 16 * kGqULd + 16 * kGqRows;
constexpr int kGqHLd = kGqPanel * kGqGroup + 4;
constexpr int kGqXLd = kGqGroup + 4;
constexpr int kGqX = kGqRows * kGqHLd;                              // a group's values, [row][column]
constexpr int kGqD = kGqX + kGqRows * kGqXLd;                       // two groups' 16 x 16 diagonal blocks, [c][j % 4][j / 4]
constexpr int kGqInv = kGqD + 2 * kGqGroup * kGqChunk;              // two groups' 1 / U[c,c], 64 bits
constexpr int kGqPanelLds = kGqInv + 2 * kGqGroup * 2;
static_assert(2 * kGqStage <= kGqD && kGqPanel * kGqGroup * kGqRows <= kGqX, "what is there throughout stays so");

// One panel of up to four groups for 32 rows.  FIRST: the values come from the bf16 matrix itself (nothing behind the first panel
// has been corrected yet), so the working copy is never filled by a pass of its own.
// Wavefronts 0 and 1 do the chains, 16 rows each; 2 and 3 meanwhile take the errors of the group before from the panel's last two groups,
// and between two chains those of that group from the next one.
// Bound: the chain of 64 dependent quantise-and-correct steps per group, 70 ns each, and the products between groups; the rest of the
// launch's work runs beside it.  Four lanes share a row (two: 3 % more for the whole sweep, though fewer instructions); the chain corrects
// 16 columns only (four a lane: as few as its own latency covers, and a quarter of the reads of U from LDS), the group's later
// columns get those 16 errors as matrix products.  14336 rows, us: alone (the last panel) 21 for the values (7 of matrix instructions a
// workgroup, 448 workgroups) and 6.5 a group; beside the rest 35 and 14, the vector instructions and the fp32 matrix
// instructions taking their time from each other.
// HALVES (no more than two groups): two wavefronts share a group's values, 16 rows each (8000 x 320 42.0 -> 38.6 us, 4096 x 384 46.7 -> 43.2).
template <int BITS, bool FIRST, bool HALVES>
__device__ __forceinline__ void gq_panel_rows(float* s_all, const uint16_t* __restrict__ w, float* v, const float* __restrict__ u, long N, long K,
                                              long base, int n_groups, const GqErr& before, const GqErr& err, bool corrections, bool last, bool spread,
                                              uint8_t* __restrict__ codes, uint16_t* __restrict__ scale, uint16_t* __restrict__ zero)
{
#pragma clang fp contract(off)
    constexpr int qmax = (1 << BITS) - 1;
    constexpr int n_words = kGqGroup * BITS / 32;               // 16 (int8), 8 (int4), 4 (int2)
    float* const s_e = s_all;                                   // errors, [column][row], negated
    float* const s_x = s_all + kGqX;
    float* const s_d = s_all + kGqD;
    double* const s_inv = reinterpret_cast<double*>(s_all + kGqInv);
    // spread: the chains (wavefronts 0 and 1 of what follows) on the workgroup's first and third
    const int tid = spread ? (threadIdx.x & 63) | (threadIdx.x & 64) << 1 | (threadIdx.x & 128) >> 1 : threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rg = lane >> 4, cl = lane & 15;
    const long block = blockIdx.x, row0 = block * kGqRows;
    // ---- the values, a group a wavefront or two, minus the errors of the panel before.
    // Register i of tile (t, x): row r16 + 16 t + 4 rg + i, column 4 cl + x.
    {
        constexpr int kTiles = HALVES ? 1 : 2;
        const int group = HALVES ? wave >> 1 : wave, r16 = HALVES ? 16 * (wave & 1) : 0;
        f32x4_t acc[kTiles][4];
        if (group < n_groups) {
#pragma unroll
            for (int t = 0; t < kTiles; t++)
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const long row = min(row0 + r16 + 16 * t + 4 * rg + i, N - 1);  // rows past the last one redo it and keep the result to themselves
                    const long at = row * K + base + kGqGroup * group + 4 * cl;
                    float4 val;
                    if constexpr (FIRST) {
                        const uint2 raw = load_global<uint2>(w + at);
                        val = make_float4(bf16_lo(raw.x), bf16_hi(raw.x), bf16_lo(raw.y), bf16_hi(raw.y));
                    } else {
                        val = load_global<float4>(v + at);
                    }
                    acc[t][0][i] = val.x; acc[t][1][i] = val.y; acc[t][2][i] = val.z; acc[t][3][i] = val.w;
                }
        }
        if (corrections) {
            long ld;
            const float* const eb = gq_err_block(before, block, ld);
            const float* const ub = u + (base - before.cols) * K + base;        // (a row's 256 floats may run over the end of U's columns, into its next row)
            const uint32_t lds = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) float*)s_all;
            auto copy = [&](int c0, int buf) {
#pragma unroll
                for (int i = 0; i < 4; i++)
                    lds_copy16((const char*)(ub + (long)(c0 + 4 * wave + i) * K), lane * 16, lds + (buf * kGqStage + (4 * wave + i) * kGqULd) * 4);
                if (wave < 2)
                    lds_copy16((const char*)eb, (uint32_t)gq_err_at(before, ld, c0 + 8 * wave + (lane >> 3), 4 * (lane & 7)) * 4,
                               lds + (buf * kGqStage + 16 * kGqULd + 8 * wave * kGqRows) * 4);
            };
            copy(0, 0);
            wait_lds_copies<0>();
            __syncthreads();
            for (int c0 = 0, buf = 0; c0 < before.cols; c0 += 16, buf ^= 1) {
                if (c0 + 16 < before.cols) copy(c0 + 16, buf ^ 1);              // (that buffer's last readers passed the barrier before)
                if (group < n_groups) {
                    const float* const sb = s_all + buf * kGqStage + rg * kGqULd + kGqGroup * group + 4 * cl;
                    const float* const sa = s_all + buf * kGqStage + 16 * kGqULd + rg * kGqRows + r16 + cl;
#pragma unroll
                    for (int kk = 0; kk < 4; kk++) {
                        const float4 b4 = *reinterpret_cast<const float4*>(sb + 4 * kk * kGqULd);
                        float a[kTiles];
#pragma unroll
                        for (int t = 0; t < kTiles; t++) a[t] = sa[4 * kk * kGqRows + 16 * t];
                        const float b[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
                        for (int t = 0; t < kTiles; t++)
#pragma unroll
                            for (int x = 0; x < 4; x++) acc[t][x] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t], b[x], acc[t][x], 0, 0, 0);
                    }
                }
                wait_lds_copies<0>();
                __syncthreads();
            }
        }
        if (group < n_groups) {
#pragma unroll
            for (int t = 0; t < kTiles; t++)
#pragma unroll
                for (int i = 0; i < 4; i++)
                    *reinterpret_cast<float4*>(s_all + (r16 + 16 * t + 4 * rg + i) * kGqHLd + kGqGroup * group + 4 * cl) =
                        make_float4(acc[t][0][i], acc[t][1][i], acc[t][2][i], acc[t][3][i]);
        }
    }
    const bool chain = wave < 2;
    const int cw = wave - 2;                                    // wavefronts 2 and 3: half of every group's columns
    // the diagonal of U for a group's chain, by wavefronts 2 and 3
    auto diagonal = [&](int g) {
        const long first = base + kGqGroup * g;
        const int at0 = tid - 128;
        if (at0 < kGqGroup) s_inv[(g & 1) * kGqGroup + at0] = 1.0 / (double)u[(first + at0) * K + first + at0];
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int at = at0 + 128 * h, c = at >> 2, i = at & 3;
            const float4 d = load_global<float4>(u + (first + c) * K + first + (c & ~15) + 4 * i);
            float* const dst = s_d + (g & 1) * kGqGroup * kGqChunk + c * kGqChunk + i;
            dst[0] = d.x; dst[4] = d.y; dst[8] = d.z; dst[12] = d.w;
        }
    };
    // the panel's later groups, o = 0: the next one.  Register i of tile (t, x): row 16 t + 4 rg + i, column 32 cw + 2 cl + x
    f32x4_t rest[3][2][2];
    if (!chain) diagonal(0);
    __syncthreads();
    if (!chain) {
#pragma unroll
        for (int h = 0; h < 4; h++) {
            const int at = tid - 128 + 128 * h, row = at >> 4, c = 4 * (at & 15);
            *reinterpret_cast<float4*>(s_x + row * kGqXLd + c) = *reinterpret_cast<const float4*>(s_all + row * kGqHLd + c);
        }
#pragma unroll
        for (int o = 0; o < 3; o++)
            if (1 + o < n_groups)
#pragma unroll
                for (int t = 0; t < 2; t++)
#pragma unroll
                    for (int i = 0; i < 4; i++) {
                        const float2 val = *reinterpret_cast<const float2*>(s_all + (16 * t + 4 * rg + i) * kGqHLd + kGqGroup * (1 + o) + 32 * cw + 2 * cl);
                        rest[o][t][0][i] = val.x;
                        rest[o][t][1][i] = val.y;
                    }
    }
    __syncthreads();                                            // the values have been read: errors may take their place
    long eld;
    float* const eb = gq_err_block(err, block, eld);
    float2 ub[16];
    // rows of group g of U, this lane's two columns of group `of`
    auto fetch = [&](int g, int of) {
        const float* const from = u + (base + kGqGroup * g + rg) * K + base + kGqGroup * of + 32 * cw + 2 * cl;
#pragma unroll
        for (int kk = 0; kk < 16; kk++) ub[kk] = load_global<float2>(from + (long)(4 * kk) * K);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto correct = [&](f32x4_t (&c)[2][2], int g) {
        const float* const ap = s_e + (kGqGroup * g + rg) * kGqRows + cl;
#pragma unroll
        for (int kk = 0; kk < 16; kk++) {
            const float a[2] = {ap[4 * kk * kGqRows], ap[4 * kk * kGqRows + 16]};
#pragma unroll
            for (int t = 0; t < 2; t++) {
                c[t][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t], ub[kk].x, c[t][0], 0, 0, 0);
                c[t][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t], ub[kk].y, c[t][1], 0, 0, 0);
            }
        }
    };
    if (chain) {
#pragma unroll 1
        for (int g = 0; g < n_groups; g++) {
            const int r = lane >> 2, q = lane & 3;              // the chain's layout: row r, columns 4 m + q
            const long row = row0 + 16 * wave + r;
            float* const sx = s_x + 16 * wave * kGqXLd;         // this wavefront's own from here on
            float* const se = s_e + kGqGroup * g * kGqRows + 16 * wave;
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
            float x[16];
#pragma unroll
            for (int m = 0; m < 16; m++) x[m] = sx[r * kGqXLd + 4 * m + q];
            f32x4_t later[3];                                   // the pieces behind the first, in the matrix instructions' layout
#pragma unroll
            for (int tt = 1; tt < 4; tt++)
#pragma unroll
                for (int i = 0; i < 4; i++) later[tt - 1][i] = sx[(4 * rg + i) * kGqXLd + 16 * tt + cl];
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
            const _Float16 zh = (_Float16)lo;                   // round to nearest even
            const float range = hi - lo;
            const float step = range / (float)qmax;             // correctly rounded division
            const _Float16 sh = (_Float16)step;
            const float m = (float)zh, s = (float)sh;
            const float inv = (s > 0.0f) ? (1.0f / s) : 0.0f;
            uint32_t words[n_words];
            auto emit = [&](int k, float ne) { se[(4 * k + q) * kGqRows + r] = ne; };      // the errors of columns 4 k .. 4 k + 3, this lane's 4 k + q
            // Sixteen columns by the chain, then their products onto the pieces behind them, errors ascending as the chain would
            // have applied them.
            float piece[4] = {x[0], x[1], x[2], x[3]};
            const double* const si = s_inv + (g & 1) * kGqGroup;
            const float* const sd = s_d + (g & 1) * kGqGroup * kGqChunk;
            auto carry = [&](auto from) {
                constexpr int T = decltype(from)::value, first = T == 0 ? 0 : T == 1 ? 12 : 20;
                const float* const ap = se + (16 * T + rg) * kGqRows + cl;
                float a[4];
#pragma unroll
                for (int kk = 0; kk < 4; kk++) a[kk] = ap[4 * kk * kGqRows];
#pragma unroll
                for (int tt = T + 1; tt < 4; tt++) {
#pragma unroll
                    for (int kk = 0; kk < 4; kk++)
                        later[tt - 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[kk], between[first + 4 * (tt - T - 1) + kk], later[tt - 1], 0, 0, 0);
                    if (tt == T + 1) {
#pragma unroll
                        for (int i = 0; i < 4; i++) sx[(4 * rg + i) * kGqXLd + 16 * tt + cl] = later[tt - 1][i];
#pragma unroll
                        for (int i = 0; i < 4; i++) piece[i] = sx[r * kGqXLd + 16 * tt + 4 * i + q];
                    }
                }
            };
            bool subnormal = gq_chunk_chain<BITS, 0>(piece, q, m, s, inv, sd, si, words, emit);
            carry(std::integral_constant<int, 0>());
            subnormal |= gq_chunk_chain<BITS, 16>(piece, q, m, s, inv, sd, si, words, emit);
            carry(std::integral_constant<int, 1>());
            subnormal |= gq_chunk_chain<BITS, 32>(piece, q, m, s, inv, sd, si, words, emit);
            carry(std::integral_constant<int, 2>());
            subnormal |= gq_chunk_chain<BITS, 48>(piece, q, m, s, inv, sd, si, words, emit);
            if (__any(subnormal)) {
#pragma unroll
                for (int m2 = 0; m2 < 16; m2++) sx[r * kGqXLd + 4 * m2 + q] = x[m2];
                gq_group_chain_exact<BITS>(sx, r, q, m, s, inv, ud, K, words, emit);
            }
            if (row < N) {
                uint8_t* dst = codes + (row * K + base + kGqGroup * g) * BITS / 8;
                constexpr int mine = n_words / 4;               // each lane of a quad writes a quarter of the row's codes
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
            __syncthreads();                                    // the group's errors are there
            __syncthreads();                                    // ... and the next one's values
        }
        return;
    }
#pragma unroll 1
    for (int g = 0; g < n_groups; g++) {
        if (g > 0) {
            // group g - 1's errors from the groups behind the present one, and to memory for the next launch
#pragma unroll
            for (int o = 0; o < 2; o++)
                if (g + 1 + o < n_groups) {
                    fetch(g - 1, g + 1 + o);
                    correct(rest[o], g - 1);
                }
            if (!last)
#pragma unroll
                for (int h = 0; h < 4; h++) {
                    const int at = tid - 128 + 128 * h, c = kGqGroup * (g - 1) + (at >> 3), r = 4 * (at & 7);
                    store_global(eb + gq_err_at(err, eld, c, r), *reinterpret_cast<const float4*>(s_e + c * kGqRows + r));
                }
        }
        if (g + 1 < n_groups) {
            diagonal(g + 1);
            fetch(g, g + 1);
        }
        __syncthreads();                                        // the group's errors are there
        if (g + 1 < n_groups) {
            correct(rest[0], g);
#pragma unroll
            for (int t = 0; t < 2; t++)
#pragma unroll
                for (int i = 0; i < 4; i++)
                    *reinterpret_cast<float2*>(s_x + (16 * t + 4 * rg + i) * kGqXLd + 32 * cw + 2 * cl) = make_float2(rest[0][t][0][i], rest[0][t][1][i]);
#pragma unroll
            for (int o = 0; o < 2; o++)
#pragma unroll
                for (int t = 0; t < 2; t++) {
                    rest[o][t][0] = rest[o + 1][t][0];
                    rest[o][t][1] = rest[o + 1][t][1];
                }
        }
        __syncthreads();                                        // ... and the next one's values
    }
    if (!last) {
        const int g = n_groups - 1;
#pragma unroll
        for (int h = 0; h < 4; h++) {
            const int at = tid - 128 + 128 * h, c = kGqGroup * g + (at >> 3), r = 4 * (at & 7);
            store_global(eb + gq_err_at(err, eld, c, r), *reinterpret_cast<const float4*>(s_e + c * kGqRows + r));
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
// lane's own place (c = rg, row or column 4 cl); lda8, ldb8: eight c's further.  values() requests acc's values, behind the first operands.
template <typename Values>
__device__ __forceinline__ void gq_tile_products(GqTile& acc, float* s_op, int wave, const float* ap, long lda8, const float* bp, long ldb8, int n,
                                                 Values values)
{
    constexpr int kStage = 2 * 16 * kGqGroup;                   // floats of one operand
    const int lane = threadIdx.x & 63;
    float* const put = s_op + (wave & 1) * 16 * kGqGroup + (wave >> 1) * 4 * kGqGroup + 4 * lane;
    const float* const get_a = s_op + (wave >> 1) * 16 * kGqGroup + 4 * lane;
    const float* const get_b = s_op + kStage + (wave & 1) * 16 * kGqGroup + 4 * lane;
    float4 fa[2], fb[2];
    auto fetch = [&] {
        fa[0] = load_global<float4>(ap);
        fa[1] = load_global<float4>(ap + lda8);
        fb[0] = load_global<float4>(bp);
        fb[1] = load_global<float4>(bp + ldb8);
        ap += 2 * lda8;
        bp += 2 * ldb8;
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
    values();
    __builtin_amdgcn_sched_barrier(0);
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

// v[r, j] = fma(-E[c, r], U[c, j], v[r, j]) for the columns c of the panel before in ascending order, every row r, columns
// [col_begin, K).  A wavefront owns 64 x 64 values, a workgroup 128 x 128; FIRST: v's values are still those of w.
// Bound: fp32 matrix instructions (a register-only loop holds 150 TFLOP/s; with operands from LDS and barriers 148).  Behind 14336 rows
// 256 columns more cost 17 us = 110 TFLOP/s, 120 without the chains beside them; the values' way in and out is 6 % of it.
template <bool FIRST>
__device__ __forceinline__ void gq_rest(float* s_op, const uint16_t* __restrict__ w, float* v, const float* __restrict__ u, long N, long K, long base,
                                        const GqErr& err, long col_begin, uint32_t wg)
{
    constexpr int kRows = 2 * kGqRows;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rg = lane >> 4, cl = lane & 15;
    // Workgroups are dealt to the eight XCDs in turn: an XCD takes every eighth pair of row blocks, and walks them eight
    // pairs at a time across all columns, so that the 64 tiles it runs at a time share 8 row and 8 column operands in its L2.
    const uint32_t row_pairs = (uint32_t)((N + 2 * kRows - 1) / (2 * kRows));
    const uint32_t col_pairs = (uint32_t)((K - col_begin + 2 * kGqGroup - 1) / (2 * kGqGroup));
    const uint32_t xcd = wg & 7, at = wg >> 3;
    const uint32_t per_xcd = (row_pairs + 7) >> 3;
    const uint32_t band = at / (8 * col_pairs), in_band = at - band * 8 * col_pairs;
    const uint32_t height = min(8u, per_xcd - 8 * band);
    const uint32_t cp = in_band / height, rp = xcd + 8 * (8 * band + in_band - cp * height);
    if (rp >= row_pairs) return;
    // a wavefront whose block lies outside (an odd number of blocks) works on the last one as well and keeps it to itself
    const long n_blocks = (N + kRows - 1) / kRows;
    const long block = min(2 * (long)rp + (wave >> 1), n_blocks - 1);
    const long col0 = min(col_begin + (2 * (long)cp + (wave & 1)) * kGqGroup, K - kGqGroup);
    const bool mine = 2 * (long)rp + (wave >> 1) == block && col_begin + (2 * (long)cp + (wave & 1)) * kGqGroup == col0;
    const long row0 = block * kRows;
    const bool whole = row0 + kRows <= N;
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
    auto values = [&] {
        if (whole) {
#pragma unroll
            for (int r = 0; r < 16; r++) load(r >> 2, r & 3, src + r * K + off);
        } else {
            const int last = (int)(N - 1 - row0);
#pragma unroll
            for (int r = 0; r < 16; r++) load(r >> 2, r & 3, src + min(16 * rg + r, last) * K + 4 * cl);
        }
    };
    // the errors of 64 rows are two blocks': lanes with cl < 8 read the first one's
    const long e_blocks = (N + kGqRows - 1) / kGqRows;
    long eld;
    const float* const eb = gq_err_block(err, min(2 * min(2 * (long)rp + (wave & 1), n_blocks - 1) + (cl >> 3), e_blocks - 1), eld);
    const int per = err.cols >> 5;                              // columns c a row of the errors, 8 or 4
    gq_tile_products(acc, s_op, wave, eb + gq_err_at(err, eld, 4 * (wave >> 1) + rg, 4 * (cl & 7)), per == 8 ? eld : 2 * eld,
                     u + (base + 4 * (wave >> 1) + rg) * K + col0 + 4 * cl, 8 * K, err.cols, values);
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

// The same corrections where those workgroups leave the chip half empty (one takes 15 us of matrix instructions whatever
// there is beside it): a workgroup 64 x 64, a wavefront 32 x 32, the operands of 64 columns c at a time through LDS.  Up to three
// quarters of a workgroup of the other kind per compute unit.
template <bool FIRST>
__device__ __forceinline__ void gq_rest_small(float* s_a, const uint16_t* __restrict__ w, float* v, const float* __restrict__ u, long N, long K,
                                              long base, const GqErr& err, long col_begin, uint32_t wg)
{
    constexpr int kRows = 2 * kGqRows;
    float* const s_b = s_a + kGqGroup * kGqGroup;               // errors, rows of U: [c][64]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rg = lane >> 4, cl = lane & 15, wi = wave >> 1, wj = wave & 1;
    const uint32_t n_blocks = (uint32_t)((N + kRows - 1) / kRows);
    const long cb = wg / n_blocks, block = wg - (uint32_t)cb * n_blocks;
    const long col0 = col_begin + cb * kGqGroup, row0 = block * kRows;
    long eld;
    const long e_blocks = (N + kGqRows - 1) / kGqRows;
    const float* const eb = gq_err_block(err, min(2 * block + ((tid & 15) >> 3), e_blocks - 1), eld);
    float4 sa[4], sb[4];
    auto fetch = [&](int c0) {
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int c = c0 + (tid >> 4) + 16 * i;
            sa[i] = load_global<float4>(eb + gq_err_at(err, eld, c, 4 * (tid & 7)));
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
    for (int c0 = 0; c0 < err.cols; c0 += kGqGroup) {
        if (c0 > 0) __syncthreads();                    // the operands before have been read
#pragma unroll
        for (int i = 0; i < 4; i++) {
            *reinterpret_cast<float4*>(s_a + 4 * (tid + 256 * i)) = sa[i];
            *reinterpret_cast<float4*>(s_b + 4 * (tid + 256 * i)) = sb[i];
        }
        __syncthreads();
        fetch(min(c0 + kGqGroup, err.cols - kGqGroup));  // (past the end: the last ones again, unused)
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

// A panel's launch: its rows first, 32 a workgroup, so that the chains start at once, then the columns behind it.
// FIRST: the values of both are still those of w (the first two panels).
// The whole sweep, us, with the panel's rows (64 a workgroup) and the columns behind it in launches of their own / so: 14336 x 4096
// 2525 / 2340, 4096 x 4096 1166 / 944, 8000 x 1024 208 / 165, 2500 x 2048 391 / 325, 200 x 4096 588 / 548, 14336 x 512 90 / 87.
enum GqBehind { kGqNothing, kGqSmall, kGqLarge };        // columns behind: none and no more than two groups in the panel; 64 x 64, 128 x 128 a workgroup
template <int BITS, bool FIRST, GqBehind BEHIND>
__global__ __launch_bounds__(256, 3) void gptq_panel_kernel(const uint16_t* __restrict__ w, float* v, const float* __restrict__ u, long N, long K,
                                                            long base, int n_groups, GqErr before, GqErr err, int row_blocks, int spread,
                                                            uint8_t* __restrict__ codes, uint16_t* __restrict__ scale, uint16_t* __restrict__ zero)
{
    __shared__ __attribute__((aligned(16))) float s_all[kGqPanelLds];
    static_assert(kGqPanelLds >= 2 * 2 * 2 * 16 * kGqGroup, "the other workgroups' operands fit");
    const long next = base + kGqGroup * n_groups;
    if ((int)blockIdx.x < row_blocks)
        gq_panel_rows<BITS, FIRST, BEHIND == kGqNothing>(s_all, w, v, u, N, K, base, n_groups, before, err, base > 0, next >= K, spread, codes, scale, zero);
    else if constexpr (BEHIND == kGqSmall)
        gq_rest_small<FIRST>(s_all, w, v, u, N, K, base - before.cols, before, next, blockIdx.x - row_blocks);
    else if constexpr (BEHIND == kGqLarge)
        gq_rest<FIRST>(s_all, w, v, u, N, K, base - before.cols, before, next, blockIdx.x - row_blocks);
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

// x of lane N of every row of sixteen lanes, to the row's sixteen lanes
template <int N>
__device__ __forceinline__ float row_bcast(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x150 + N, 0xF, 0xF, true));
}

// a[J + i] = fma(x of lane J + i of the row of sixteen, y, a[J + i]), i = 0 .. N - 1: the broadcast is part of the multiply-add, which the
// compiler makes two instructions of.  (The waits: a value that is read across lanes must be two wait states old.)
#define DYMOE_FMAC_BCAST(A_, I_) "v_fmac_f32_dpp %[" #A_ "], %[x], %[y] row_newbcast:%[" #I_ "] row_mask:0xf bank_mask:0xf\n\t"
template <int J, int N>
__device__ __forceinline__ void gq_fmac_bcast(float (&a)[16], float x, float y)
{
    if constexpr (N >= 7) {
        asm("s_nop 1\n\t" DYMOE_FMAC_BCAST(a0, j0) DYMOE_FMAC_BCAST(a1, j1) DYMOE_FMAC_BCAST(a2, j2)
            DYMOE_FMAC_BCAST(a3, j3) DYMOE_FMAC_BCAST(a4, j4) DYMOE_FMAC_BCAST(a5, j5)
            DYMOE_FMAC_BCAST(a6, j6)
            : [a0] "+&v"(a[J]), [a1] "+&v"(a[J + 1]), [a2] "+&v"(a[J + 2]), [a3] "+&v"(a[J + 3]), [a4] "+&v"(a[J + 4]),
              [a5] "+&v"(a[J + 5]), [a6] "+&v"(a[J + 6])
            : [x] "v"(x), [y] "v"(y), [j0] "n"(J), [j1] "n"(J + 1), [j2] "n"(J + 2), [j3] "n"(J + 3), [j4] "n"(J + 4), [j5] "n"(J + 5),
              [j6] "n"(J + 6));
        gq_fmac_bcast<J + 7, N - 7>(a, x, y);
    } else if constexpr (N >= 4) {
        asm("s_nop 1\n\t" DYMOE_FMAC_BCAST(a0, j0) DYMOE_FMAC_BCAST(a1, j1) DYMOE_FMAC_BCAST(a2, j2)
            DYMOE_FMAC_BCAST(a3, j3)
            : [a0] "+&v"(a[J]), [a1] "+&v"(a[J + 1]), [a2] "+&v"(a[J + 2]), [a3] "+&v"(a[J + 3])
            : [x] "v"(x), [y] "v"(y), [j0] "n"(J), [j1] "n"(J + 1), [j2] "n"(J + 2), [j3] "n"(J + 3));
        gq_fmac_bcast<J + 4, N - 4>(a, x, y);
    } else if constexpr (N >= 2) {
        asm("s_nop 1\n\t" DYMOE_FMAC_BCAST(a0, j0) DYMOE_FMAC_BCAST(a1, j1) "s_nop 1"
            : [a0] "+&v"(a[J]), [a1] "+&v"(a[J + 1])
            : [x] "v"(x), [y] "v"(y), [j0] "n"(J), [j1] "n"(J + 1));
        gq_fmac_bcast<J + 2, N - 2>(a, x, y);
    } else if constexpr (N >= 1) {
        asm("s_nop 1\n\t" DYMOE_FMAC_BCAST(a0, j0) "s_nop 1"
            : [a0] "+&v"(a[J])
            : [x] "v"(x), [y] "v"(y), [j0] "n"(J));
        gq_fmac_bcast<J + 1, N - 1>(a, x, y);
    }
}
#undef DYMOE_FMAC_BCAST

// The Cholesky factor of the 16 x 16 block whose row lane % 16 the lane holds, by one wavefront (its four rows of sixteen lanes do
// the same): pivots and multipliers through the data-parallel primitives, which the multiply-adds take as operands.  a: the row,
// replaced by the factor's (what stands right of the diagonal is worth nothing).
// Column C's chain is pivot, estimate, root, quotient, column C + 1; the column before goes to the other columns meanwhile.
template <int C>
__device__ __forceinline__ void gq_chol_column(float (&a)[16], float less_before, float before)
{
    // square root and quotient: the hardware's estimate of 1 / sqrt(d) and one residual step each (finite operands; see
    // the step kernel for infinite ones)
    const float d = row_bcast<C>(a[C]);
    const float y = __builtin_amdgcn_rsqf(d);
    if constexpr (C > 0 && C < 15) {
        gq_fmac_bcast<C + 1, 15 - C>(a, less_before, before);
        __builtin_amdgcn_sched_barrier(0);
    }
    const float s0 = d * y, l0 = a[C] * y;
    const float sq = __builtin_fmaf(__builtin_fmaf(-s0, s0, d), 0.5f * y, s0);
    const float l = __builtin_fmaf(__builtin_fmaf(-sq, l0, a[C]), y, l0);
    const float less = -l;
    if constexpr (C < 15) a[C + 1] = __builtin_fmaf(row_bcast<C + 1>(less), l, a[C + 1]);
    a[C] = ((threadIdx.x & 15) == C) ? sq : l;
    if constexpr (C < 15) gq_chol_column<C + 1>(a, less, l);
}

// Piece p of the diagonal block in LDS (rows and columns 16 p .. 16 p + 15, row stride kGqLd) becomes its Cholesky factor, by one
// wavefront; also as the solving wavefronts read it (s_q[c][row % 4][row / 4]) and its diagonal with the reciprocals.
constexpr int kGqLd = kGqGroup + 4;
__device__ __forceinline__ void gq_chol_piece(float* s_m, int p, float* s_q, float2* s_inv)
{
    const int lane = threadIdx.x & (kWave - 1), row = lane & 15;
    float* const own = s_m + (16 * p + row) * kGqLd + 16 * p;
    float a[16], dg;
    auto diagonal = [&] {
        dg = a[0];
#pragma unroll
        for (int c = 1; c < 16; c++) dg = (row == c) ? a[c] : dg;
    };
#pragma unroll
    for (int c = 0; c < 4; c++) {
        const float4 t = *reinterpret_cast<const float4*>(own + 4 * c);
        a[4 * c] = t.x; a[4 * c + 1] = t.y; a[4 * c + 2] = t.z; a[4 * c + 3] = t.w;
    }
    gq_chol_column<0>(a, 0.0f, 0.0f);
    diagonal();
    if (!__all(dg > 1e-15f && dg < 1e15f)) {
        // a pivot so large or small that the estimate's steps may leave the range (or none at all: NaN): root and division as
        // they are, in LDS (the wavefront's rows of lanes write the same values)
#pragma unroll 1
        for (int c = 0; c < 16; c++) {
            const float root = sqrtf(s_m[(16 * p + c) * kGqLd + 16 * p + c]);
            const float l = (row == c) ? root : own[c] / root;
            own[c] = l;
            for (int j = c + 1; j < 16; j++) own[j] = __builtin_fmaf(-l, s_m[(16 * p + j) * kGqLd + 16 * p + c], own[j]);
        }
#pragma unroll
        for (int c = 0; c < 16; c++) a[c] = own[c];
        diagonal();
    }
    if (lane < 16) {
#pragma unroll
        for (int c = 0; c < 4; c++) *reinterpret_cast<float4*>(own + 4 * c) = make_float4(a[4 * c], a[4 * c + 1], a[4 * c + 2], a[4 * c + 3]);
#pragma unroll
        for (int c = 0; c < 16; c++) s_q[(16 * p + c) * kGqChunk + (row & 3) * 4 + (row >> 2)] = a[c];
        s_inv[16 * p + row] = make_float2(dg, 1.0f / dg);
    }
}

// One 16 x 16 tile loses the products of 16 columns c, ascending: acc[row, col] = fma(-x[row, c], y[col, c], acc[row, col]).  x: where
// lane (rg, cl) finds -x[row cl, c = rg], x_step: four columns further; y likewise (y[col cl, c = rg]), row stride kGqLd.
__device__ __forceinline__ void gq_tile_less(f32x4_t& acc, const float* x, int x_step, float sign, const float* y)
{
    float xv[4], yv[4];
#pragma unroll
    for (int kk = 0; kk < 4; kk++) {
        xv[kk] = sign * x[kk * x_step];
        yv[kk] = y[4 * kk];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kk = 0; kk < 4; kk++) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(xv[kk], yv[kk], acc, 0, 0, 0);
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
// block and out of its own block of v, makes the diagonal block's Cholesky factor and substitutes.
// The others bring the rest of v forward, steps in pairs (a panel: steps 2 q and 2 q + 1), so that a block of v is read and
// written once per panel:
//   k = 2 q + 2   panel q into the block pairs q + 1 and q + 2 (columns and rows) and into some of the blocks behind them
//   k = 2 q + 3   panel q into the other blocks; step 2 q + 2 alone into block row and column 2 q + 4, which step 2 q + 4 needs
// A workgroup takes more than half of a compute unit's LDS and so has it to itself: beside tiles a solver took 3.5 us longer.
// The launch lasts as long as the solver's chain (11 us and 2.3 to the next launch), or, for the first steps of a large K, as the tiles.
// K = 4096: 1345 -> 1160 us, 1024: 259 -> 212, 256: 65 -> 54 (with solvers beside three tiles on a compute unit, step k - 1's products in
// front of the chain, and a lane per row in the piece's factor).  Beyond 5120 columns the tiles are all there is, and one workgroup of them on a
// unit is as good as three small ones only while its rounds are whole and its operands come from its XCD's L2: with a panel's
// tiles split for whole rounds (gptq_steps.hpp) and neighbouring blocks on one XCD 4096: 1138 -> 1112 us, 6144 2790 -> 2668 (three
// small ones 2825), 8192 5619 -> 5474 (5539), 14336 25.65 -> 25.21 ms (25.49).
// The quotient is the product with the reciprocal and one residual step.  For finite operands that differs from a division
// in the last place at most; an infinite operand or quotient gives NaN where the division gives infinity, but it has no
// place in a positive definite matrix: what it is subtracted from, a later pivot, becomes NaN either way.
constexpr int kGqStepThreads = 512;
constexpr int kGqTileLds = 3 * kGqGroup * kGqGroup;                 // floats: a tile's operands of 64 columns c, one of two buffers
constexpr int kGqPLd = kGqGroup + 16;                               // row stride of P's blocks in the solver: c and c + 1 on other banks

// The tiles' part of a launch: 64 x 128 block rows of tiles dealt out to the workers, of whom those behind the first `early` start when a
// solver has left them a compute unit (kGqSkip blocks later).  32 x 32 of a block a wavefront; the operands of 64 columns c at a
// time go straight to LDS, and they and the next block's values are on their way while the products before run.
// Bound: fp32 matrix instructions, 3.6 us a block at 2.27 GHz; 4.4 to 5.4 measured, and 2.5 to start.  (Through registers, operands read from LDS where
// they are used: 6.2.)
__device__ __forceinline__ void gq_step_tiles(float* s_all, float* v, long K, int k, const float* slots, const GqWide& wide, int worker,
                                              int workers, int early, int blocks)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rg = lane >> 4, cl = lane & 15, wi = wave >> 2, wq = wave & 3;
    const int last = (int)(K / kGqGroup) - 1, q = (int)wide.q, n_single = (k & 1) ? (int)wide.single : 0;
    struct Block {
        int ib, sj, jb, s0;
        bool single, mine;
    };
    auto locate = [&](int at, Block& b) {                           // false: nothing to do there (the same in the whole workgroup)
        b.single = at < n_single;
        if (b.single) {
            const int below = last - k;
            b.ib = at < below ? k + 1 + at : k + 1;
            b.sj = at < below ? q + 2 : at - below;
        } else {
            // (block row k, the upper half of the pairs si = q + 1, is the solvers')
            const int below = (int)wide.pairs - q - 1, upper = 2 * below - 1;
            int half = at - n_single, si;
            if (!(k & 1) && half < upper) {
                half++;
                si = q + 1 + (half >> 1);
                b.sj = q + 1;
            } else if (!(k & 1) && half < upper + q + 1) {
                b.sj = half - upper;
                si = q + 1;
                half = 1;
            } else {
                if (!(k & 1)) half += 2 * (int)wide.pairs - upper - (q + 1);
                const int tile = half >> 1;
                if (!(k & 1) && tile < (int)wide.near) {
                    if (tile < (int)wide.pairs + below - 1) { si = q + 2 + tile - (int)wide.pairs; b.sj = q + 2; }
                    else { si = q + 2; b.sj = tile - (int)wide.pairs - (below - 1); }
                } else {
                    // m = si - 1 column pairs (without q + 1 and q + 2) of every pair si >= q + 3
                    const int r = ((k & 1) ? tile + (int)wide.first : tile - (int)wide.near) + (q + 2) * (q + 1) / 2;
                    int m = (int)((sqrtf(8.0f * (float)r + 1.0f) + 1.0f) * 0.5f);
                    while (m * (m - 1) / 2 > r) m--;
                    while ((m + 1) * m / 2 <= r) m++;
                    si = m + 1;
                    b.sj = r - m * (m - 1) / 2;
                    if (b.sj >= q + 1) b.sj += 2;
                }
            }
            b.ib = 2 * si + (half & 1);
        }
        b.s0 = b.single ? k - 1 : 2 * q;
        b.jb = min(2 * b.sj + (wq >> 1), last);
        b.mine = 2 * b.sj + (wq >> 1) <= last && b.jb <= b.ib &&
                 (b.single ? b.jb == k + 1 || (b.ib == k + 1 && b.jb != k) : b.jb != b.s0 + 2);
        return b.ib <= last;
    };
    int round = worker < early ? 0 : kGqSkip;
    auto next = [&](Block& b) {                                     // false: no block is left
        for (;;) {
            const int at = round < kGqSkip ? round * early + worker : kGqSkip * early + (round - kGqSkip) * workers + worker;
            if (at >= blocks) return false;
            round++;
            if (locate(at, b)) return true;
        }
    };
    // a step's operands: rows [c][64] and two column blocks [c][64] each, straight to LDS
    const uint32_t lds = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) float*)s_all;
    auto copy = [&](const Block& b, int s, int buf) {
        const uint32_t to = lds + (buf * kGqTileLds + wave * 4 * kGqGroup) * 4;
#pragma unroll
        for (int o = 0; o < 3; o++) {
            long ld;
            const char* const from = (const char*)gq_p_block(v, K, slots, s, o == 0 ? b.ib : min(2 * b.sj + o - 1, last), ld);
            const uint32_t row = (uint32_t)ld * 4, at = (4 * wave + rg) * row + cl * 16;
#pragma unroll
            for (int i = 0; i < 2; i++)
                lds_copy16(from + (long)(32 * i) * row, at, to + (o * kGqGroup * kGqGroup + i * 32 * kGqGroup) * 4);
        }
    };
    // interleaved as in GqTile, with two row and two column tiles: register i of tile (x, y) is row 8 rg + 2 i + x, column
    // 2 cl + y
    const uint32_t off = 8 * rg * (uint32_t)K + 2 * cl;
    auto place = [&](const Block& b) { return v + ((long)b.ib * kGqGroup + 32 * wi) * K + (long)b.jb * kGqGroup + 32 * (wq & 1); };
    float2 val[8];
    auto request = [&](const Block& b) {
        const float* const src = place(b);
        const bool zero = b.jb == b.s0 || (!b.single && b.jb == b.s0 + 1);      // (block columns of the panel itself: L^-1's part starts here)
#pragma unroll
        for (int r = 0; r < 8; r++) val[r] = zero ? make_float2(0.0f, 0.0f) : load_global<float2>(src + r * K + off);
        __builtin_amdgcn_sched_barrier(0);
    };
    f32x4_t acc[2][2];                                              // negated: fma(-x, y, c) is -fma(x, y, -c)
    // operands of sixteen columns c, four a product
    float2 av[2][4], bv[2][4];
    auto read = [&](int set, int buf, int g) {
        const float* const ap = s_all + buf * kGqTileLds + (16 * g + rg) * kGqGroup + 32 * wi + 2 * cl;
        const float* const bp = s_all + buf * kGqTileLds + (1 + (wq >> 1)) * kGqGroup * kGqGroup + (16 * g + rg) * kGqGroup + 32 * (wq & 1) + 2 * cl;
#pragma unroll
        for (int kk = 0; kk < 4; kk++) {
            av[set][kk] = *reinterpret_cast<const float2*>(ap + kk * 4 * kGqGroup);
            bv[set][kk] = *reinterpret_cast<const float2*>(bp + kk * 4 * kGqGroup);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto multiply = [&](int set) {
#pragma unroll
        for (int kk = 0; kk < 4; kk++) {
            const float2 x = av[set][kk], y = bv[set][kk];
            acc[0][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.x, y.x, acc[0][0], 0, 0, 0);
            acc[0][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.x, y.y, acc[0][1], 0, 0, 0);
            acc[1][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.y, y.x, acc[1][0], 0, 0, 0);
            acc[1][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.y, y.y, acc[1][1], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // The 64 columns in buffer buf; the last sixteen's products run when the next buffer's first operands are on their way, so that
    // neither the barrier nor the reads behind it find the matrix cores idle.
    auto pass = [&](int buf, bool more) {
#pragma unroll
        for (int g = 0; g < 3; g++) {
            read((g + 1) & 1, buf, g + 1);
            multiply(g & 1);
        }
        wait_lds_copies<0>();
        __syncthreads();
        if (more) read(0, buf ^ 1, 0);                              // the same in the whole workgroup
        multiply(1);
    };
    Block b, then;
    if (!next(b)) return;
    copy(b, b.s0, 0);
    request(b);
    wait_lds_copies<0>();
    __syncthreads();
    read(0, 0, 0);
    int buf = 0;
    for (;;) {
#pragma unroll
        for (int r = 0; r < 8; r++) {
            acc[r & 1][0][r >> 1] = -val[r].x;
            acc[r & 1][1][r >> 1] = -val[r].y;
        }
        if (!b.single) {
            copy(b, b.s0 + 1, buf ^ 1);                             // (that buffer's last readers passed the barrier before)
            pass(buf, true);
            buf ^= 1;
            if (b.jb == b.s0 + 1) {                                 // ... with the panel's second step
#pragma unroll
                for (int x = 0; x < 2; x++) acc[x][0] = acc[x][1] = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
            }
        }
        const bool more = next(then);
        if (more) {
            copy(then, then.s0, buf ^ 1);
            request(then);
        }
        pass(buf, more);
        buf ^= 1;
        if (b.mine) {
            float* const dst = place(b);
#pragma unroll
            for (int r = 0; r < 8; r++) store_global(dst + r * K + off, make_float2(-acc[r & 1][0][r >> 1], -acc[r & 1][1][r >> 1]));
        }
        if (!more) return;
        b = then;
    }
}

// The solver's part: workgroup jb of step k.  Four stages of 16 columns; in each wavefront 0 factors the 16 x 16 piece on the
// diagonal, then the rows below it and the own block's columns are substituted, 16 rows a wavefront (four lanes a row).  What the
// stages' tiles need besides -- step k - 1's products, 64 columns deep, and those of the pieces before -- the other wavefronts
// do while wavefront 0 factors, each tile just in time.
//   slot (piece being factored)   wavefront 0    6                    7                    1, 2, 3, 5 (16 columns j of the own block each)
//   0                             P 00           P 10, 20, 21         P 30, 31, 11         P of columns c 0, 1
//   1                             - 11           - 21, P 22 - 22      - 31, P 32 - 32      - columns 1, P of columns 2, - columns 2
//   2                             - 22           P 33 - - 33          - 32                 - columns 2, P of columns 3, - - columns 3
//   3                             - 33                                                     - columns 3
// (P: products of step k - 1, -: of one piece before; tiles by row and column.)  Wavefront 4 shares wavefront 0's SIMD and only substitutes:
// beside matrix instructions there the factor of a piece took up to twice as long.
// Bound: the chain, us: 1.5 to start and for the operands, 1.8 the first slot, 1.3 to 1.5 the others (a factor is 440 instructions of one
// wavefront, 1.1), 1.1 a substitution.
__device__ __forceinline__ void gq_step_solve(float* s_all, float* v, long K, long k, float* slots, float* __restrict__ u, long jb)
{
    constexpr int kXLd = kGqChunk + 4;
    float* const s_p = s_all;                                       // P of step k - 1: block k, own block: [c][column]
    float* const s_m = s_p + 2 * kGqGroup * kGqPLd;                 // diagonal block, [row][column]
    float* const s_x = s_m + kGqGroup * kGqLd;                      // the own block's 16 columns of the stage, [column j][c]
    float* const s_q = s_x + kGqGroup * kXLd;                       // 16 x 16 blocks of the factor's diagonal
    float2* const s_inv = reinterpret_cast<float2*>(s_q + kGqGroup * kGqChunk);
    float* const s_e = reinterpret_cast<float*>(s_inv + kGqGroup);  // [wavefront][piece][c of the 16][column], negated
    static_assert(2 * kGqGroup * kGqPLd + kGqGroup * kGqLd + kGqGroup * kXLd + kGqGroup * kGqChunk + 2 * kGqGroup +
                      4 * 4 * kGqChunk * 16 <= 2 * kGqTileLds, "the solver's blocks fit");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rg = lane >> 4, cl = lane & 15;
    const long base = k * kGqGroup, before = k - 1;
    // rows of 16: of the own block's columns (wavefronts 1, 2, 3, 5), or of the diagonal block (4, 6, 7: rows 1, 2, 3)
    const bool own = wave == 5 || (wave >= 1 && wave <= 3);
    const int w4 = wave == 5 ? 3 : wave - 1, drow = wave == 4 ? 1 : wave - 4;
    if (wave == 0) __builtin_amdgcn_s_setprio(3);                   // the chain, beside wavefronts that only add work
    // the operands, requested at once (the workgroups of the launch before left them in other L2s, a microsecond away) ...
    const bool with_own = jb != k && k > 0;
    float4 stage[2][2];
#pragma unroll
    for (int b = 0; b < 2; b++)
        if (k > 0 && (b == 0 || with_own)) {
            long ld;
            const float* const from = gq_p_block(v, K, slots, before, b ? jb : k, ld) + (tid >> 4) * ld + 4 * (tid & 15);
#pragma unroll
            for (int i = 0; i < 2; i++) stage[b][i] = load_global<float4>(from + 32 * i * ld);
        }
    // ... and the values of the wavefront's tiles, register i of lane (rg, cl): row 4 rg + i, column cl
    f32x4_t acc[4];
    // wavefront 0: tile 00 of the diagonal block; 6: 10, 20, 21, 22, 33; 7: 30, 31, 11, 32
    f32x4_t more;
    auto diag_tile = [&](f32x4_t& c, int row, int col) {
#pragma unroll
        for (int i = 0; i < 4; i++) c[i] = load_global<float>(v + (base + 16 * row + 4 * rg + i) * K + base + 16 * col + cl);
    };
    if (own) {
#pragma unroll
        for (int t = 0; t < 4; t++) {
            // [column j][c]: above the diagonal (rows j of v) as it lies, below it transposed
            if (jb == k) {
#pragma unroll
                for (int i = 0; i < 4; i++) acc[t][i] = (16 * w4 + 4 * rg + i == 16 * t + cl) ? 1.0f : 0.0f;
            } else if (jb == before) {                              // (L^-1's part starts with its own step)
                acc[t] = (f32x4_t){0.0f, 0.0f, 0.0f, 0.0f};
            } else if (jb > k) {
#pragma unroll
                for (int i = 0; i < 4; i++)
                    acc[t][i] = load_global<float>(v + (jb * kGqGroup + 16 * w4 + 4 * rg + i) * K + base + 16 * t + cl);
            } else {
                const float4 col = load_global<float4>(v + (base + 16 * t + cl) * K + jb * kGqGroup + 16 * w4 + 4 * rg);
                acc[t][0] = col.x; acc[t][1] = col.y; acc[t][2] = col.z; acc[t][3] = col.w;
            }
        }
    } else if (wave == 0) {
        diag_tile(acc[0], 0, 0);
    } else if (wave == 6) {
        diag_tile(acc[0], 1, 0);
        diag_tile(acc[1], 2, 0);
        diag_tile(acc[2], 2, 1);
        diag_tile(acc[3], 2, 2);
        diag_tile(more, 3, 3);
    } else if (wave == 7) {
        diag_tile(acc[0], 3, 0);
        diag_tile(acc[1], 3, 1);
        diag_tile(acc[2], 1, 1);
        diag_tile(acc[3], 3, 2);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (k > 0) {
#pragma unroll
        for (int b = 0; b < 2; b++)
#pragma unroll
            for (int i = 0; i < 2; i++)
                *reinterpret_cast<float4*>(s_p + b * kGqGroup * kGqPLd + ((tid >> 4) + 32 * i) * kGqPLd + 4 * (tid & 15)) = stage[b][i];
    }
    __syncthreads();
    // step k - 1's products: rows from block `block` (0: k, 1: own) of P, columns from block k
    auto products = [&](f32x4_t& c, int block, int row, int col) {
        if (k == 0 || (block == 1 && jb == k)) return;              // the same in the whole workgroup
        const float* const ap = s_p + block * kGqGroup * kGqPLd + rg * kGqPLd + 16 * row + cl;
        const float* const bp = s_p + rg * kGqPLd + 16 * col + cl;
        float x[16], y[16];
#pragma unroll
        for (int kk = 0; kk < 16; kk++) {
            x[kk] = ap[4 * kk * kGqPLd];
            y[kk] = bp[4 * kk * kGqPLd];
        }
        __builtin_amdgcn_sched_barrier(0);                          // all of them requested before the first is waited for
        c = -c;                                                     // (fma(-x, y, c) is -fma(x, y, -c))
#pragma unroll
        for (int kk = 0; kk < 16; kk++) c = __builtin_amdgcn_mfma_f32_16x16x4f32(x[kk], y[kk], c, 0, 0, 0);
        c = -c;
    };
    auto put = [&](const f32x4_t& c, int row, int col) {            // a tile of the diagonal block
#pragma unroll
        for (int i = 0; i < 4; i++) s_m[(16 * row + 4 * rg + i) * kGqLd + 16 * col + cl] = c[i];
    };
    auto less = [&](f32x4_t& c, int row, int col, int piece) {      // ... loses a piece's products
        gq_tile_less(c, s_m + (16 * row + cl) * kGqLd + 16 * piece + rg, 4, -1.0f, s_m + (16 * col + cl) * kGqLd + 16 * piece + rg);
    };
    float* const se = s_e + w4 * 4 * kGqChunk * 16;
    auto own_less = [&](f32x4_t& c, int col, int piece) {
        gq_tile_less(c, se + piece * kGqChunk * 16 + lane, 64, 1.0f, s_m + (16 * col + cl) * kGqLd + 16 * piece + rg);
    };
    const int rr = lane >> 2, q = lane & 3;                         // substitution: four lanes per row
    const long j = jb * kGqGroup + 16 * w4 + rr;
    float* const pj = jb == k ? slots + k * kGqGroup * kGqGroup + q * kGqGroup + 16 * w4 + rr : v + (base + q) * K + j;
    const long pld = jb == k ? kGqGroup : K;
    float* const uj = u + (K - 1 - base - q) * K + (K - 1 - j);
#pragma unroll
    for (int s = 0; s < 4; s++) {
        // ---- the slot
        if (own) {
            if (s == 0) products(acc[0], 1, w4, 0);
            else own_less(acc[s], s, s - 1);
#pragma unroll
            for (int i = 0; i < 4; i++) s_x[(16 * w4 + 4 * rg + i) * kXLd + cl] = acc[s][i];
            if (s < 3) {
                products(acc[s + 1], 1, w4, s + 1);
#pragma unroll
                for (int p = 0; p < s; p++) own_less(acc[s + 1], s + 1, p);
            }
        } else if (wave == 0) {
            if (s == 0) {
                products(acc[0], 0, 0, 0);
            } else {
#pragma unroll
                for (int i = 0; i < 4; i++) acc[0][i] = s_m[(16 * s + 4 * rg + i) * kGqLd + 16 * s + cl];
                less(acc[0], s, s, s - 1);
            }
            put(acc[0], s, s);
            gq_chol_piece(s_m, s, s_q, s_inv);
        } else if (wave == 6) {
            // (the diagonal's next tile goes to LDS once wavefront 0 has only its last piece to take off)
            if (s == 0) {
                products(acc[0], 0, 1, 0);
                put(acc[0], 1, 0);
                products(acc[1], 0, 2, 0);
                put(acc[1], 2, 0);
                products(acc[2], 0, 2, 1);
            } else if (s == 1) {
                less(acc[2], 2, 1, 0);
                put(acc[2], 2, 1);
                products(acc[3], 0, 2, 2);
                less(acc[3], 2, 2, 0);
                put(acc[3], 2, 2);
            } else if (s == 2) {
                products(more, 0, 3, 3);
                less(more, 3, 3, 0);
                less(more, 3, 3, 1);
                put(more, 3, 3);
            }
        } else if (wave == 7) {
            if (s == 0) {
                products(acc[0], 0, 3, 0);
                put(acc[0], 3, 0);
                products(acc[2], 0, 1, 1);
                put(acc[2], 1, 1);
                products(acc[1], 0, 3, 1);
            } else if (s == 1) {
                less(acc[1], 3, 1, 0);
                put(acc[1], 3, 1);
                products(acc[3], 0, 3, 2);
                less(acc[3], 3, 2, 0);
            } else if (s == 2) {
                less(acc[3], 3, 2, 1);
                put(acc[3], 3, 2);
            }
        }
        __syncthreads();
        // ---- substitution
        if (own || (wave >= 4 && drow > s)) {
            float* const xr = own ? s_x + (16 * w4 + rr) * kXLd : s_m + (16 * drow + rr) * kGqLd + 16 * s;
            float x[4], keep = 0.0f;
#pragma unroll
            for (int i = 0; i < 4; i++) x[i] = xr[4 * i + q];
            const float4* const sd = reinterpret_cast<const float4*>(s_q + 16 * s * kGqChunk + 4 * q);
            float4 d[kGqChunk];
            float2 dg[kGqChunk];
#pragma unroll
            for (int i = 0; i < kGqChunk; i++) {
                d[i] = sd[i * (kGqChunk / 4)];
                dg[i] = s_inv[16 * s + i];
            }
#pragma unroll
            for (int i = 0; i < kGqChunk; i++) {
                const int k4 = i / 4, c = i % 4;
                const float xi = c == 0 ? quad_bcast<0>(x[k4]) : c == 1 ? quad_bcast<1>(x[k4]) : c == 2 ? quad_bcast<2>(x[k4]) : quad_bcast<3>(x[k4]);
                const float e0 = xi * dg[i].y;
                const float e = __builtin_fmaf(__builtin_fmaf(-dg[i].x, e0, xi), dg[i].y, e0);    // the quotient: one residual step
                keep = (q == c) ? e : keep;
                if (c == 3) {
                    if (own) {
                        pj[(long)(16 * s + 4 * k4) * pld] = keep;
                        uj[-(long)(16 * s + 4 * k4) * K] = (jb > k) ? 0.0f : keep;
                        se[s * kGqChunk * 16 + (4 * k4 + q) * 16 + rr] = -keep;
                    } else {
                        xr[4 * k4 + q] = keep;
                    }
                }
                const float dd[4] = {d[i].x, d[i].y, d[i].z, d[i].w};
#pragma unroll
                for (int m = (c == 3) ? k4 + 1 : k4; m < 4; m++) x[m] = __builtin_fmaf(-e, dd[m], x[m]);
            }
        }
        if (s < 3) __syncthreads();
    }
}

// A workgroup's place in the order of the blocks.  Workgroups are handed to the eight XCDs in turn: neighbouring blocks, which share their
// rows' operands, go to one XCD's, so that its L2 fetches them once (11008 columns 12.40 -> 12.20 ms, 2048 445 -> 434 us).
__device__ __forceinline__ int gq_worker(int w, int workers, int early)
{
    const int first = w < early ? 0 : early, n = (w < early ? min(early, workers) : workers) - first;
    const int xcd = (w - first) & 7;
    return first + xcd * (n >> 3) + min(xcd, n & 7) + ((w - first) >> 3);
}

__global__ __launch_bounds__(kGqStepThreads, 2) void gptq_step_kernel(float* v, long K, long k, float* slots, float* __restrict__ u,
                                                                     GqWide wide, int early, int blocks)
{
    __shared__ __attribute__((aligned(16))) float s_all[2 * kGqTileLds];
    static_assert(sizeof(s_all) > 80 * 1024, "one workgroup per compute unit");
    const int nb = (int)(K / kGqGroup);
    if ((int)blockIdx.x < nb) gq_step_solve(s_all, v, K, k, slots, u, blockIdx.x);
    else gq_step_tiles(s_all, v, K, (int)k, slots, wide, gq_worker((int)blockIdx.x - nb, (int)gridDim.x - nb, early), (int)gridDim.x - nb, early, blocks);
}

// The sweep over up to kGqMostRows rows, a launch a panel; v: their place in the working copy.
constexpr long kGqMostRows = 1L << 28;
static int gq_sweep(dymoe_ctx* ctx, const uint16_t* w, const float* u, long N, long K, int bits, uint8_t* codes, uint16_t* sc, uint16_t* zr,
                    float* v, float* tail, hipStream_t st)
{
    const long row_blocks = gq_row_blocks(N);
    const int panel = gq_panel(N), cols = panel * kGqGroup;
    GqErr before = {};
    for (long base = 0; base < K; base += cols) {
        const long left = (K - base) / kGqGroup;
        const int groups = (int)(left < panel ? left : panel);
        const long next = base + groups * kGqGroup;
        const GqErr err = {v + base, tail + ((base / cols) & 1) * cols * kGqRows, K, N / kGqRows, cols};
        const GqBehindGrid behind = gq_behind_grid(N, K, base, next, ctx->num_cu);
        const long rest = behind.workgroups;
        const bool first = base <= cols;
        // A workgroup's wavefronts begin one SIMD on from the one's before it on the compute unit: with both chains on neighbouring wavefronts,
        // two workgroups on a unit have two chains on one SIMD.  us, neighbours / spread: 14336 x 64 8.4 / 7.0, x 256 30.2 / 28.2, x 1024 229 / 226, 18000 x
        // 1024 297 / 278.  Beside more columns than are resident, or with several rounds of row blocks, they are as good or better together
        // (12289 x 4096 2148 / 2163, 57344 x 512 243 / 247).
        const bool spread = row_blocks > ctx->num_cu && row_blocks <= 4L * ctx->num_cu && rest <= 3L * ctx->num_cu;
        auto go = [&](auto kernel) {
            dymoe_launch(ctx, rest ? DYMOE_K_GPTQ_TRAIL : DYMOE_K_GPTQ_GROUP, kernel, dim3((unsigned)(row_blocks + rest)), dim3(256), 0, st, w, v,
                         u, N, K, base, groups, before, err, (int)row_blocks, (int)spread, codes, sc, zr);
        };
        auto pick = [&](auto bits) {
            constexpr int BITS = decltype(bits)::value;
            if (next >= K && groups <= 2) first ? go(gptq_panel_kernel<BITS, true, kGqNothing>) : go(gptq_panel_kernel<BITS, false, kGqNothing>);
            else if (behind.small) first ? go(gptq_panel_kernel<BITS, true, kGqSmall>) : go(gptq_panel_kernel<BITS, false, kGqSmall>);
            else first ? go(gptq_panel_kernel<BITS, true, kGqLarge>) : go(gptq_panel_kernel<BITS, false, kGqLarge>);
        };
        if (bits == 8) pick(std::integral_constant<int, 8>());
        else if (bits == 4) pick(std::integral_constant<int, 4>());
        else pick(std::integral_constant<int, 2>());
        DYMOE_HIP_LAUNCH_CHECK();
        before = err;
    }
    return DYMOE_OK;
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
    float* v = reinterpret_cast<float*>(workspace);
    float* tail = reinterpret_cast<float*>((char*)workspace + gq_round256((size_t)N * (size_t)K * 4));
    // A dimension of a launch holds fewer than 2^32 threads, a workgroup of 256 takes 32 rows, and rows are independent: 2^28 at a
    // time.  (Only the last of them can be ragged: the buffer for its errors is one.)
    for (long row = 0; row < N; row += kGqMostRows) {
        const int rc = gq_sweep(ctx, (const uint16_t*)w_bf16 + row * K, u, N - row < kGqMostRows ? N - row : kGqMostRows, K, bits,
                                codes + row * K * bits / 8, (uint16_t*)scale + row * (K / kGqGroup), (uint16_t*)zero + row * (K / kGqGroup),
                                v + row * K, tail, (hipStream_t)stream);
        if (rc != DYMOE_OK) return rc;
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
        const GqWide wide = gq_wide(nb, k, ctx->num_cu);
        const long blocks = gq_wide_blocks(wide, k), workers = gq_workers(nb, ctx->num_cu, blocks);
        dymoe_launch(ctx, DYMOE_K_GPTQ_FACTOR, gptq_step_kernel, dim3((unsigned)(nb + workers)), dim3(kGqStepThreads), 0, st, v, K, k, slots, u,
                     wide, (int)gq_early(nb, ctx->num_cu), (int)blocks);
        DYMOE_HIP_LAUNCH_CHECK();
    }
    return DYMOE_OK;
}

}  // extern "C"
