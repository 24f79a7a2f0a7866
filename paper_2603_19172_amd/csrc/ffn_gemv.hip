// Decode path of the mixed-precision SwiGLU expert FFN: bandwidth-bound
// dequant-fused GEMV in two launches: phase 1 (gate and up projections, SwiGLU;
// one (token, expert) pair per grid row) and phase 2 (down projection of every
// expert of a token, weighted by the gate and summed into y).
//
// A wavefront streams weight rows.  A row is cut into segments of 2048
// columns; in a segment every lane owns a fixed set of 32 columns, so the
// activations a lane needs never change while it streams rows: they are
// loaded once into registers (packed pairs) and the weight stream is the only
// memory traffic of the loop.
//   bf16 rows : 4 x 16-byte loads per lane and segment, bf16 dot2 (phase 1)
//               or fp32 FMA (phase 2, fp32 intermediate)
//   int8 rows : two 16-byte loads per lane and segment (32 codes = half a group)
//   int4 rows : one 16-byte load per lane and segment (32 codes = half a group)
//   int2 rows : one  8-byte load per lane and segment (32 codes = half a group)
// The row loop is software pipelined: the loads of the next batch of rows are
// issued before the current batch is reduced, and every load is unconditional
// (lanes past the end of a row re-read the row's tail against zero
// activations) so that the loop body is straight-line code.
//
// Quantised codes are turned into fp16 without integer->float conversions:
// OR-ing a code field into the mantissa of 2^n (n chosen so that the field's
// lowest bit weighs 1) gives the fp16 number 2^n + q.  The dot product with
// the activations then runs on fp16 dot2 (fp32 accumulate) and the 2^n * x
// terms are removed with one precomputed constant per lane:
//   sum_k (s q_k + m) x_k = s * (sum_k (2^n_k + q_k) x_k - sum_k 2^n_k x_k) + m * sum_k x_k.
#include <math.h>

#include <type_traits>

#include "common.hpp"
#include "assign.hpp"
#include "ffn_layout.hpp"
#include "norm_device.hpp"
#include "route_device.hpp"

namespace dymoe {

constexpr int kGvThreads = 256;
constexpr int kGvWaves = kGvThreads / kWave;

// ------------------------------------------------------------------ activations

// 32 activations of one lane (quantised layouts), as fp16 pairs ordered for
// the code extraction below, plus the two per-lane constants.
struct LaneX {
    uint32_t r[16];
    float xsum;  // sum of the 64 activations of the lane's quantisation group (the lane's 32 and its partner's)
    float xoff;  // sum of 2^n_k * x_k
};

__device__ __forceinline__ float h2f(_Float16 h) { return (float)h; }

// v[32] are the lane's activations in column order.
template <int BITS>
__device__ __forceinline__ void arrange_lane_x(const float* v, LaneX& lx)
{
    _Float16 hv[32];
    float sum = 0.0f;
#pragma unroll
    for (int i = 0; i < 32; i++) {
        hv[i] = (_Float16)v[i];
        sum += h2f(hv[i]);
    }
    lx.xsum = sum + dpp_get<0xB1, 0xF>(sum);       // quad_perm [1,0,3,2]: lanes 2i and 2i+1 share a group
    float off = 0.0f;
    if (BITS == 8) {
        // dword d holds codes 4d..4d+3, one per byte; pairs (b0,b1) and (b2,b3), all offset by 1024
#pragma unroll
        for (int i = 0; i < 16; i++) {
            half2_t pr = {hv[2 * i], hv[2 * i + 1]};
            lx.r[i] = __builtin_bit_cast(uint32_t, pr);
        }
        off = 1024.0f * sum;
    } else if (BITS == 4) {
        // dword d holds codes 8d..8d+7 in nibbles 0..7
        // pairs: (n0,n4)+1024, (n1,n5)+64, (n2,n6)+1024, (n3,n7)+64
#pragma unroll
        for (int d = 0; d < 4; d++) {
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const _Float16 a = hv[8 * d + j], b = hv[8 * d + 4 + j];
                half2_t pr = {a, b};
                lx.r[4 * d + j] = __builtin_bit_cast(uint32_t, pr);
                const float wgt = (j & 1) ? 64.0f : 1024.0f;
                off += wgt * (h2f(a) + h2f(b));
            }
        }
    } else {
        // dword d holds codes 16d..16d+15 in 2-bit fields 0..15; pair j = (field j, field 8+j)
        // offsets by field position: 1024, 256, 64, 16, 4, then (after >>10) 1024, 256, 64
        const float wgt[8] = {1024.0f, 256.0f, 64.0f, 16.0f, 4.0f, 1024.0f, 256.0f, 64.0f};
#pragma unroll
        for (int d = 0; d < 2; d++) {
#pragma unroll
            for (int j = 0; j < 8; j++) {
                const _Float16 a = hv[16 * d + j], b = hv[16 * d + 8 + j];
                half2_t pr = {a, b};
                lx.r[8 * d + j] = __builtin_bit_cast(uint32_t, pr);
                off += wgt[j] * (h2f(a) + h2f(b));
            }
        }
    }
    lx.xoff = off;
}

// sum_k (2^n_k + q_k) x_k over the lane's 32 int4 codes (one uint4)
__device__ __forceinline__ float dot_q4(const uint4 c, const LaneX& lx)
{
    const uint32_t w[4] = {c.x, c.y, c.z, c.w};
    float acc = 0.0f;
#pragma unroll
    for (int d = 0; d < 4; d++) {
        const uint32_t v = w[d], v8 = w[d] >> 8;
        acc = dot2_f16(and_or(v, 0x000F000Fu, 0x64006400u), lx.r[4 * d + 0], acc);
        acc = dot2_f16(and_or(v, 0x00F000F0u, 0x54005400u), lx.r[4 * d + 1], acc);
        acc = dot2_f16(and_or(v8, 0x000F000Fu, 0x64006400u), lx.r[4 * d + 2], acc);
        acc = dot2_f16(and_or(v8, 0x00F000F0u, 0x54005400u), lx.r[4 * d + 3], acc);
    }
    return acc;
}

// the same over the lane's 32 int2 codes (one uint2)
__device__ __forceinline__ float dot_q2(const uint2 c, const LaneX& lx)
{
    const uint32_t w[2] = {c.x, c.y};
    float acc = 0.0f;
#pragma unroll
    for (int d = 0; d < 2; d++) {
        const uint32_t v = w[d], v10 = w[d] >> 10;
        acc = dot2_f16(and_or(v, 0x00030003u, 0x64006400u), lx.r[8 * d + 0], acc);
        acc = dot2_f16(and_or(v, 0x000C000Cu, 0x5C005C00u), lx.r[8 * d + 1], acc);
        acc = dot2_f16(and_or(v, 0x00300030u, 0x54005400u), lx.r[8 * d + 2], acc);
        acc = dot2_f16(and_or(v, 0x00C000C0u, 0x4C004C00u), lx.r[8 * d + 3], acc);
        acc = dot2_f16(and_or(v, 0x03000300u, 0x44004400u), lx.r[8 * d + 4], acc);
        acc = dot2_f16(and_or(v10, 0x00030003u, 0x64006400u), lx.r[8 * d + 5], acc);
        acc = dot2_f16(and_or(v10, 0x000C000Cu, 0x5C005C00u), lx.r[8 * d + 6], acc);
        acc = dot2_f16(and_or(v10, 0x00300030u, 0x54005400u), lx.r[8 * d + 7], acc);
    }
    return acc;
}

// the same over the lane's 32 int8 codes (two uint4): a byte b becomes the fp16 number 1024 + b
__device__ __forceinline__ float dot_q8(const uint4 c0, const uint4 c1, const LaneX& lx)
{
    const uint32_t w[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
    float acc = 0.0f;
#pragma unroll
    for (int d = 0; d < 8; d++) {
        acc = dot2_f16(__builtin_amdgcn_perm(0x64646464u, w[d], 0x04010400u), lx.r[2 * d], acc);
        acc = dot2_f16(__builtin_amdgcn_perm(0x64646464u, w[d], 0x04030402u), lx.r[2 * d + 1], acc);
    }
    return acc;
}

// activations of one lane for bf16 rows: NSEG x 4 chunks of 8, packed bf16 pairs
template <int NSEG>
struct LaneXB {
    uint4 r[NSEG][4];
};

// ------------------------------------------------------------------ weight rows

struct ExpertMat {
    const uint16_t* w;      // bf16
    const uint8_t* q;       // packed codes at the expert's precision
    const uint16_t* s;      // fp16 scale
    const uint16_t* z;      // fp16 zero
};

__device__ __forceinline__ ExpertMat pick_mat(const dymoe_expert_fmt& ex, int mat, int b)
{
    ExpertMat m;
    m.w = reinterpret_cast<const uint16_t*>(ex.w[mat]);
    if (b == 8) {
        m.q = ex.q8[mat];
        m.s = reinterpret_cast<const uint16_t*>(ex.s8[mat]);
        m.z = reinterpret_cast<const uint16_t*>(ex.z8[mat]);
    } else if (b == 4) {
        m.q = ex.q4[mat];
        m.s = reinterpret_cast<const uint16_t*>(ex.s4[mat]);
        m.z = reinterpret_cast<const uint16_t*>(ex.z4[mat]);
    } else {
        m.q = ex.q2[mat];
        m.s = reinterpret_cast<const uint16_t*>(ex.s2[mat]);
        m.z = reinterpret_cast<const uint16_t*>(ex.z2[mat]);
    }
    return m;
}

// Whether the table held the pointers of this matrix at b bits.  The bit widths are chosen on the device, so only the
// kernels can tell that an assigned format is absent; they test exactly the pointers they are about to read through.
__device__ __forceinline__ bool mat_present(const ExpertMat& m, int b)
{
    return (b == 16) ? (m.w != nullptr) : (m.q != nullptr && m.s != nullptr && m.z != nullptr);
}

// What the second phase reads of a (token, expert) pair: its down projection, its gate weight and its bit width (0: the pair
// adds nothing).  Left in the workspace by the first phase's workgroup that has the pair's first rows: read from the pair's
// index on, expert, bit width and table entry are three loads that wait for each other, and the whole second phase is a few of
// those long where the experts are small.
struct alignas(32) PairDown {
    const void* codes;      // bf16 rows where bits == 16
    const uint16_t* s;
    const uint16_t* z;
    float gate;
    int32_t bits;
};
static_assert(sizeof(PairDown) == 32, "one scalar load");

// (called by the workgroup with the pair's first rows; a format that is not in the table leaves the pair out)
__device__ __forceinline__ void leave_pair_down(PairDown* __restrict__ down, const ExpertMat& m2, int p, int b, float gate,
                                                unsigned* __restrict__ flags)
{
    if (threadIdx.x != 0) return;
    const bool there = mat_present(m2, b);
    if (!there) atomicOr(flags, DYMOE_FLAG_FORMAT_MISSING);
    PairDown d;
    d.codes = b == 16 ? (const void*)m2.w : (const void*)m2.q;
    d.s = m2.s;
    d.z = m2.z;
    d.gate = gate;
    d.bits = there ? b : 0;
    down[p] = d;
}

// what one lane loads of one row: NSEG segments starting at column seg0 * 2048
template <int BITS, int NSEG> struct RowRegs;
template <int NSEG> struct RowRegs<16, NSEG> { uint4 c[NSEG][4]; };      // (the first NCH of 4, see load_row)
template <int NSEG> struct RowRegs<4, NSEG> { uint4 c[NSEG]; uint16_t sz[NSEG]; };
template <int NSEG> struct RowRegs<2, NSEG> { uint2 c[NSEG]; uint16_t sz[NSEG]; };
template <int NSEG> struct RowRegs<8, NSEG> { uint4 c[NSEG][2]; uint16_t sz[NSEG]; };

// Issue the loads of row `row` (K columns).  Lanes past the end of the row
// re-read its tail: finite weights against zero activations add nothing.
// Weights are read once per step: where a load instruction covers whole cache
// lines (consecutive lanes, consecutive 16 or 8 bytes) it is marked non-temporal.
// NCH: how many of a bf16 segment's four 512-column chunks the rows reach into.
template <int BITS, int NSEG, int NCH = 4>
__device__ __forceinline__ void load_row(const ExpertMat& m, long row, int K, int seg0, int lane,
                                         RowRegs<BITS, NSEG>& rr)
{
    if constexpr (BITS == 16) {
        const uint16_t* base = m.w + row * K;
#pragma unroll
        for (int s = 0; s < NSEG; s++)
#pragma unroll
            for (int j = 0; j < NCH; j++) {
                const int col = min((seg0 + s) * kSeg + (j * kWave + lane) * 8, K - 8);
                rr.c[s][j] = load_global_nt<uint4>(base + col);
            }
    } else {
        const long G = K >> 6;
        const uint8_t* codes = m.q + row * ((long)K * BITS / 8);
#pragma unroll
        for (int s = 0; s < NSEG; s++) {
            const int col0 = min((seg0 + s) * kSeg + 32 * lane, K - 32);
            if constexpr (BITS == 8) {
                // (ordinary loads: the two pieces of a lane interleave with its neighbours', and only a
                // cached line serves both)
                rr.c[s][0] = load_global<uint4>(codes + col0);
                rr.c[s][1] = load_global<uint4>(codes + col0 + 16);
            } else if constexpr (BITS == 4) rr.c[s] = load_global_nt<uint4>(codes + (col0 >> 1));
            else rr.c[s] = load_global_nt<uint2>(codes + (col0 >> 2));
            // the two lanes of a group share its scale and zero: the even lane fetches the scale, the odd one the
            // zero (one load instruction for both; dot_row_q puts the halves together)
            rr.sz[s] = load_global<uint16_t>(((lane & 1) ? m.z : m.s) + row * G + (col0 >> 6));
        }
    }
}

// per-lane partial dot product of a loaded quantised row
template <int BITS, int NSEG>
__device__ __forceinline__ float dot_row_q(const RowRegs<BITS, NSEG>& rr, const LaneX (&lx)[NSEG])
{
    float part = 0.0f;
#pragma unroll
    for (int s = 0; s < NSEG; s++) {
        float acc;
        if constexpr (BITS == 8) acc = dot_q8(rr.c[s][0], rr.c[s][1], lx[s]);
        else if constexpr (BITS == 4) acc = dot_q4(rr.c[s], lx[s]);
        else acc = dot_q2(rr.c[s], lx[s]);
        // group total = scale * sum_k q_k x_k + zero * sum_k x_k over both lanes' halves: the even lane, which holds
        // the scale, takes the first term (its partner's sum comes over by DPP), the odd lane the second
        const float qx = acc - lx[s].xoff;
        const float qx_group = qx + dpp_get<0xB1, 0xF>(qx);
        const float coef = h2f(f16_from_bits(rr.sz[s]));
        part += coef * ((threadIdx.x & 1) ? lx[s].xsum : qx_group);
    }
    return part;
}

// bf16 row against bf16 activations (exact products, fp32 accumulation)
template <int NSEG>
__device__ __forceinline__ float dot_row_b(const RowRegs<16, NSEG>& rr, const LaneXB<NSEG>& lx)
{
    float a = 0.0f;
#pragma unroll
    for (int s = 0; s < NSEG; s++)
#pragma unroll
        for (int j = 0; j < 4; j++) {
            a = dot2_bf16(rr.c[s][j].x, lx.r[s][j].x, a);
            a = dot2_bf16(rr.c[s][j].y, lx.r[s][j].y, a);
            a = dot2_bf16(rr.c[s][j].z, lx.r[s][j].z, a);
            a = dot2_bf16(rr.c[s][j].w, lx.r[s][j].w, a);
        }
    return a;
}

// ---------------------------------------------------------------- phase 1
// h[p,f] = silu(W1[f,:] . x_t) * (W3[f,:] . x_t)
// A wavefront takes RF consecutive f per iteration (2*RF rows in flight).

template <int BITS> struct Phase1Rows { static constexpr int RF = (BITS == 16) ? 1 : (BITS == 2 ? 4 : 2); };

// arrange() makes the activations of what was requested before: the first rows are on their way when it waits for them.
template <int BITS, int NSEG, typename ArrangeFn, typename DotFn>
__device__ __forceinline__ void phase1_rows(const ExpertMat& m1, const ExpertMat& m3, int H,
                                            int f_begin, int f_end, float* __restrict__ hrow,
                                            ArrangeFn arrange, DotFn dot)
{
    constexpr int RF = Phase1Rows<BITS>::RF;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    // two register sets used in turn (the loop body handles two batches), so that a batch requested one pass
    // ahead is consumed where it landed: no copying from a "next" set to a "current" one
    RowRegs<BITS, NSEG> ra[2 * RF], rb[2 * RF];
    int f = f_begin + wave * RF;
    if (f >= f_end) return;
    constexpr int kStep = kGvWaves * RF;
    auto fetch = [&](RowRegs<BITS, NSEG>(&dst)[2 * RF], int f0) {   // rows clamped to the block's last row
#pragma unroll
        for (int i = 0; i < RF; i++) {
            const int fi = min(f0 + i, f_end - 1);
            load_row<BITS, NSEG>(m1, fi, H, 0, lane, dst[2 * i]);
            load_row<BITS, NSEG>(m3, fi, H, 0, lane, dst[2 * i + 1]);
        }
    };
    fetch(ra, f);
    __builtin_amdgcn_sched_barrier(0);
    const auto lx = arrange();
    auto finish = [&](const RowRegs<BITS, NSEG>(&src)[2 * RF], int f0) {
        float a[RF], g[RF];
#pragma unroll
        for (int i = 0; i < RF; i++) {
            a[i] = dot(src[2 * i], lx);
            g[i] = dot(src[2 * i + 1], lx);
        }
#pragma unroll
        for (int i = 0; i < RF; i++) {
            a[i] = wave_sum_dpp(a[i]);
            g[i] = wave_sum_dpp(g[i]);
        }
        // lane i writes row f0 + i
        float hv = 0.0f;
#pragma unroll
        for (int i = 0; i < RF; i++)
            if (lane == i) hv = a[i] / (1.0f + __expf(-a[i])) * g[i];
        if (lane < RF && f0 + lane < f_end) hrow[f0 + lane] = hv;
    };
    if constexpr (BITS >= 8) {
        for (; f < f_end; f += 2 * kStep) {
            fetch(rb, f + kStep);                    // next batch first
            finish(ra, f);
            if (f + kStep >= f_end) break;           // the same in every lane of the wavefront
            fetch(ra, f + 2 * kStep);
            finish(rb, f + kStep);
        }
    } else {
        // int4 / int2: four and eight rows per batch make the doubled loop body long enough to cost more in
        // instruction fetch than the copies it saves (measured: 24.5 against 22.6 us on the int2 pair)
        for (; f < f_end; f += kStep) {
            fetch(rb, f + kStep);
            finish(ra, f);
#pragma unroll
            for (int i = 0; i < 2 * RF; i++) ra[i] = rb[i];
        }
    }
}

template <int BITS, int NSEG, typename Missing>
__device__ __forceinline__ void phase1_quant(const ExpertMat& m1, const ExpertMat& m3,
                                             const uint16_t* __restrict__ xrow, int H, int f_begin,
                                             int f_end, float* __restrict__ hrow, Missing missing)
{
    const int lane = threadIdx.x & (kWave - 1);
    // (columns past the end are read as the row's first and made zero when they are used)
    uint4 raw[NSEG][4];
#pragma unroll
    for (int s = 0; s < NSEG; s++) {
        const int col0 = s * kSeg + 32 * lane;
        const uint16_t* from = xrow + (col0 < H ? col0 : 0);
#pragma unroll
        for (int c = 0; c < 4; c++) raw[s][c] = *reinterpret_cast<const uint4*>(from + 8 * c);
    }
    // (tested here and not before the loads above: the table's pointers and the activations then arrive together)
    if (!mat_present(m1, BITS) || !mat_present(m3, BITS)) return missing();
    struct Lanes {
        LaneX l[NSEG];
    };
    phase1_rows<BITS, NSEG>(m1, m3, H, f_begin, f_end, hrow, [&] {
        Lanes o;
#pragma unroll
        for (int s = 0; s < NSEG; s++) {
            const bool in = s * kSeg + 32 * lane < H;
            float v[32];
#pragma unroll
            for (int c = 0; c < 4; c++) {
                const uint32_t u[4] = {raw[s][c].x, raw[s][c].y, raw[s][c].z, raw[s][c].w};
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const uint32_t q = in ? u[i] : 0;
                    v[8 * c + 2 * i] = bf16_lo(q);
                    v[8 * c + 2 * i + 1] = bf16_hi(q);
                }
            }
            arrange_lane_x<BITS>(v, o.l[s]);
        }
        return o;
    }, [](const RowRegs<BITS, NSEG>& rr, const Lanes& o) { return dot_row_q<BITS, NSEG>(rr, o.l); });
}

template <int NSEG, typename Missing>
__device__ __forceinline__ void phase1_bf16(const ExpertMat& m1, const ExpertMat& m3,
                                            const uint16_t* __restrict__ xrow, int H, int f_begin,
                                            int f_end, float* __restrict__ hrow, Missing missing)
{
    const int lane = threadIdx.x & (kWave - 1);
    LaneXB<NSEG> raw;
#pragma unroll
    for (int s = 0; s < NSEG; s++)
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int col = s * kSeg + (j * kWave + lane) * 8;
            raw.r[s][j] = *reinterpret_cast<const uint4*>(xrow + (col < H ? col : 0));
        }
    if (!mat_present(m1, 16) || !mat_present(m3, 16)) return missing();
    phase1_rows<16, NSEG>(m1, m3, H, f_begin, f_end, hrow, [&] {
#pragma unroll
        for (int s = 0; s < NSEG; s++)
#pragma unroll
            for (int j = 0; j < 4; j++)
                if (s * kSeg + (j * kWave + lane) * 8 >= H) raw.r[s][j] = make_uint4(0, 0, 0, 0);
        return raw;
    }, [](const RowRegs<16, NSEG>& rr, const LaneXB<NSEG>& l) { return dot_row_b<NSEG>(rr, l); });
}

// One (token, expert) pair p: workgroup bx's rows of W1 and W3 of expert e at b bits
template <int NSEG>
__device__ __forceinline__ void phase1_pair(const uint16_t* __restrict__ x, const dymoe_expert_fmt* __restrict__ table, int bx,
                                            int p, int e, int b, float gate, int H, int F, int k, int rows_per_block,
                                            float* __restrict__ hbuf, PairDown* __restrict__ down, unsigned* __restrict__ flags)
{
    const int t = p / k;
    const int f_begin = bx * rows_per_block;
    const int f_end = min(F, f_begin + rows_per_block);
    const uint16_t* xrow = x + (long)t * H;
    float* hrow = hbuf + (long)p * F;
    const dymoe_expert_fmt ex = table[e];
    // The assigned format may be absent from the table: the pair then contributes nothing.  Its rows of the
    // intermediate are set to zero, so that the second phase adds nothing for it even where it finds the down projection.
    auto missing = [&]() {
        for (int f = f_begin + (int)threadIdx.x; f < f_end; f += kGvThreads) hrow[f] = 0.0f;
        if (bx == 0 && threadIdx.x == 0) atomicOr(flags, DYMOE_FLAG_FORMAT_MISSING);
    };
    if (b == 16) {
        if (bx == 0) leave_pair_down(down, pick_mat(ex, 2, 16), p, 16, gate, flags);
        phase1_bf16<NSEG>(pick_mat(ex, 0, 16), pick_mat(ex, 1, 16), xrow, H, f_begin, f_end, hrow, missing);
    } else if (b == 8) {
        if (bx == 0) leave_pair_down(down, pick_mat(ex, 2, 8), p, 8, gate, flags);
        phase1_quant<8, NSEG>(pick_mat(ex, 0, 8), pick_mat(ex, 1, 8), xrow, H, f_begin, f_end, hrow, missing);
    } else if (b == 4) {
        if (bx == 0) leave_pair_down(down, pick_mat(ex, 2, 4), p, 4, gate, flags);
        phase1_quant<4, NSEG>(pick_mat(ex, 0, 4), pick_mat(ex, 1, 4), xrow, H, f_begin, f_end, hrow, missing);
    } else {
        if (bx == 0) leave_pair_down(down, pick_mat(ex, 2, 2), p, 2, gate, flags);
        phase1_quant<2, NSEG>(pick_mat(ex, 0, 2), pick_mat(ex, 1, 2), xrow, H, f_begin, f_end, hrow, missing);
    }
}

template <int NSEG>
__global__ __launch_bounds__(kGvThreads) void gemv_phase1_kernel(
    const uint16_t* __restrict__ x, const int32_t* __restrict__ idx, const float* __restrict__ w,
    const uint8_t* __restrict__ bits, const dymoe_expert_fmt* __restrict__ table, int H, int F,
    int E, int k, int rows_per_block, float* __restrict__ hbuf, PairDown* __restrict__ down, unsigned* __restrict__ flags)
{
    // pairs in reverse: a token's later slots carry the less important experts, hence the narrower formats,
    // whose workgroups are short and latency-bound; dispatched first they overlap the wide ones instead of forming the tail
    const int p = (int)gridDim.y - 1 - (int)blockIdx.y;
    const int e = idx[p];
    const int b = (e >= 0 && e < E) ? bits[e] : 0;
    if (b != 16 && b != 8 && b != 4 && b != 2) {              // pairs of skipped experts add nothing
        if (blockIdx.x == 0 && threadIdx.x == 0) down[p].bits = 0;
        return;
    }
    phase1_pair<NSEG>(x, table, (int)blockIdx.x, p, e, b, w[p], H, F, k, rows_per_block, hbuf, down, flags);
}

// The first phase with the decode step's front end in front of it (router gating and top-k, decode importance,
// bit-width assignment: the arithmetic of dymoe_decode_front, same device functions, same order of every sum, so the
// same bits).  Every workgroup works the front end out for itself, in LDS, and goes on to its rows without a launch
// boundary and without the chain of dependent loads (pair -> expert -> bit width) the stand-alone kernel starts with;
// the first workgroup also writes the front end's outputs to memory, for the caller.  FRONT says
// where the logits come from:
//   kFrontRouter    the router's rows, read by every workgroup (64 KiB for 8 experts of 4096: from L2 by all but the first)
//   kFrontResidual  the same, of the row that residual and normalisation make of the layer before (one token): every
//                   workgroup works that out as well, while its first router rows are on their way.  As a launch of its own
//                   between two layers the step took 4.7 us of 55 (Mixtral shape, int4 experts).
//   kFrontLogits    front_logits_kernel's launch (more router rows than a workgroup reads in one trip), which takes residual
//                   and normalisation as well
// Limits (checked by the launcher): T <= kFusedMaxTokens, E <= 64 NC, k <= kFusedMaxK.
constexpr int kFusedMaxTokens = 4, kFusedMaxK = 8, kFusedMaxE = 128;
enum { kFrontRouter, kFrontResidual, kFrontLogits };

struct FusedFront {
    const uint16_t* x;        // [T,H]; kFrontResidual: the layer before's input row h
    const float* y_prev;      // kFrontResidual: ... its output, and where the normalised row goes
    float alpha;
    uint16_t* h_out;
    const uint16_t* wg;
    const float* bias;
    const float* logits;      // kFrontLogits: [T,E]
    int renorm, floor_bits;
    TierTable tiers;
    int32_t* idx;
    float* w;
    float* probs;
    float* importance;
    int32_t* load;
    uint8_t* bits;
    int32_t* rank;
};

// Logits of one token from its row in LDS (route_logits' arithmetic for TW = 1).  request() asks for what the row is made of, ahead
// of the first router rows, which come back behind it; make_row() makes the row while they are on their way.
template <int NCH, typename Request, typename MakeRow>
__device__ __forceinline__ void route_logits_of_row(const uint16_t* s_row, const uint16_t* __restrict__ wg, const float* __restrict__ bias,
                                                    int H, int E, float* logit, Request request, MakeRow make_row)
{
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    constexpr int EB = (NCH <= 8) ? 2 : 1;
    uint4 wv[EB][NCH], xr[NCH];
    auto fetch = [&](int e0) {
#pragma unroll
        for (int i = 0; i < EB; i++) {
            const uint16_t* row = wg + (size_t)min(e0 + i * kGvWaves, E - 1) * H;
#pragma unroll
            for (int c = 0; c < NCH; c++) {
                wv[i][c] = make_uint4(0, 0, 0, 0);
                if (c * kWave * 8 < H) wv[i][c] = load_global<uint4>(row + min((c * kWave + lane) * 8, H - 8));
            }
        }
    };
    request();
    __builtin_amdgcn_sched_barrier(0);
    fetch(wave);
    __builtin_amdgcn_sched_barrier(0);
    make_row();
#pragma unroll
    for (int c = 0; c < NCH; c++) {
        const int col = (c * kWave + lane) * 8;
        xr[c] = make_uint4(0, 0, 0, 0);
        if (col < H) xr[c] = *reinterpret_cast<const uint4*>(s_row + col);
    }
    for (int e0 = wave; e0 < E; e0 += kGvWaves * EB) {
        if (e0 != wave) fetch(e0);
#pragma unroll
        for (int i = 0; i < EB; i++) {
            const int e = e0 + i * kGvWaves;
            float acc = 0.0f;
#pragma unroll
            for (int c = 0; c < NCH; c++)
                if (c * kWave * 8 < H) {
                    acc = dot2_bf16(wv[i][c].x, xr[c].x, acc);
                    acc = dot2_bf16(wv[i][c].y, xr[c].y, acc);
                    acc = dot2_bf16(wv[i][c].z, xr[c].z, acc);
                    acc = dot2_bf16(wv[i][c].w, xr[c].w, acc);
                }
            const float b = (bias && e < E) ? bias[e] : 0.0f;
            const float s = wave_sum(acc);
            if (lane == 0 && e < E) logit[e] = s + b;
        }
    }
}

template <int NSEG, int NCH, int NC, int FRONT>
__global__ __launch_bounds__(kGvThreads) void decode_fused_phase1_kernel(
    const FusedFront f, const dymoe_expert_fmt* __restrict__ table, int T, int H, int F, int E, int k, int front_apart,
    int rows_per_block, float* __restrict__ hbuf, PairDown* __restrict__ down, unsigned* __restrict__ flags)
{
    __shared__ float s_logit[64 * NC];
    __shared__ float s_selp[kFusedMaxK];
    __shared__ float s_imp[64 * NC];
    __shared__ int32_t s_load[64 * NC];
    __shared__ int32_t s_idx[kFusedMaxTokens * kFusedMaxK];
    __shared__ float s_w[kFusedMaxTokens * kFusedMaxK];
    __shared__ float s_probs[kFusedMaxTokens * 64 * NC];
    __shared__ uint8_t s_bits[64 * NC];
    __shared__ int32_t s_rank[64 * NC];
    __shared__ float s_part[kNormThreads / kWave];
    __shared__ __attribute__((aligned(16))) uint16_t s_row[FRONT == kFrontResidual ? NSEG * kSeg : 8];
    const int wave = threadIdx.x / kWave;
    const bool first = blockIdx.x == 0 && blockIdx.y == 0;
    // front_apart: a workgroup of its own, the first, writes the front end's outputs, and the rest are the pairs' one after the other
    int bx = (int)blockIdx.x, pair = (int)blockIdx.y;
    if (NC > 1 && front_apart) {
        const int blocks = (F + rows_per_block - 1) / rows_per_block;
        bx--;
        pair = max(bx, 0) / blocks;
        bx -= pair * blocks;                                        // (-1: the front end's)
    }
    __builtin_assume(k >= 1 && k <= kFusedMaxK);
    for (int e = threadIdx.x; e < E; e += kGvThreads) {
        s_imp[e] = 0.0f;
        s_load[e] = 0;
    }
    for (int t = 0; t < T; t++) {
        if constexpr (FRONT == kFrontResidual) {
            // (columns past the end are read as the row's first and made zero: a load under a condition is waited for on the spot)
            uint4 h_raw[NSEG];
            float4 y_raw[NSEG][2];
            route_logits_of_row<NCH>(s_row, f.wg, f.bias, H, E, s_logit, [&] {
#pragma unroll
                for (int i = 0; i < NSEG; i++) {
                    const int j = (i * kNormThreads + (int)threadIdx.x) * 8, from = j < H ? j : 0;
                    h_raw[i] = load_global<uint4>(f.x + from);
                    y_raw[i][0] = load_global<float4>(f.y_prev + from);
                    y_raw[i][1] = load_global<float4>(f.y_prev + from + 4);
                }
            }, [&] {
                float v[NSEG][8], ss = 0.0f;
#pragma unroll
                for (int i = 0; i < NSEG; i++) {
                    residual_add(h_raw[i], y_raw[i][0], y_raw[i][1], f.alpha, v[i]);
                    const bool in = (i * kNormThreads + (int)threadIdx.x) * 8 < H;
#pragma unroll
                    for (int n = 0; n < 8; n++) v[i][n] = in ? v[i][n] : 0.0f;
                    residual_square<true>(v[i], ss);
                }
                const float inv = residual_inv_rms(ss, H, s_part);
#pragma unroll
                for (int i = 0; i < NSEG; i++) {
                    const int j = (i * kNormThreads + (int)threadIdx.x) * 8;
                    if (j < H) {
                        const uint4 o = residual_pack(v[i], inv);
                        *reinterpret_cast<uint4*>(s_row + j) = o;
                        if (first) *reinterpret_cast<uint4*>(f.h_out + j) = o;
                    }
                }
                __syncthreads();
            });
        } else if constexpr (FRONT == kFrontLogits) {
            for (int e = threadIdx.x; e < E; e += kGvThreads) s_logit[e] = f.logits[(size_t)t * E + e];
        } else {
            route_logits<1, NCH, kGvWaves>(f.x, f.wg, f.bias, T, H, E, t, s_logit);
        }
        __syncthreads();
        if (wave == 0) route_select_fixed<NC>(s_logit, s_selp, t, E, k, f.renorm, s_idx, s_w, s_probs, s_imp, s_load);
        __syncthreads();
    }
    for (int e = threadIdx.x; e < E; e += kGvThreads) {
        const float g = s_imp[e];
        s_imp[e] = (T <= 1) ? g : g / (float)T;
    }
    __syncthreads();
    const int p = T * k - 1 - pair;
    const int e = s_idx[p];
    int b = 0;
    if (first) {
        assign_all<float>(kGvThreads, E, s_imp, s_load, f.tiers, f.floor_bits, s_bits, s_rank);
        __syncthreads();
        for (int i = threadIdx.x; i < T * k; i += kGvThreads) {
            f.idx[i] = s_idx[i];
            f.w[i] = s_w[i];
        }
        if (f.probs)
            for (int i = threadIdx.x; i < T * E; i += kGvThreads) f.probs[i] = s_probs[i];
        for (int i = threadIdx.x; i < E; i += kGvThreads) {
            f.importance[i] = s_imp[i];
            f.load[i] = s_load[i];
            f.bits[i] = s_bits[i];
            if (f.rank) f.rank[i] = s_rank[i];
        }
        if (bx < 0) return;
        b = s_bits[max(e, 0)];
    } else if (e >= 0) {
        // the others need the bit width of one expert: its position is the number of lanes whose experts precede it
        const float mi = s_imp[e];
        const int ml = s_load[e];
        int pos = 0;
#pragma unroll
        for (int c = 0; c < NC; c++) {
            const int j = c * kWave + (int)(threadIdx.x & (kWave - 1));
            const float oi = s_imp[min(j, E - 1)];
            const int ol = s_load[min(j, E - 1)];
            pos += __popcll(__ballot(j < E && (oi > mi || (oi == mi && (ol > ml || (ol == ml && j < e))))));
        }
        b = tier_bits_at(pos, f.tiers, f.floor_bits);
    }
    if (e < 0 || (b != 16 && b != 8 && b != 4 && b != 2)) {
        if (bx == 0 && threadIdx.x == 0) down[p].bits = 0;
        return;
    }
    phase1_pair<NSEG>(FRONT == kFrontResidual ? s_row : f.x, table, bx, p, e, b, s_w[p], H, F, k, rows_per_block, hbuf, down, flags);
}

// ---------------------------------------------------------------- phase 2
// y[t,j] = sum_slot w[t,slot] * sum_f W2_e[j,f] * h[p,f],  p = t*k + slot, e = idx[p]
// A workgroup owns ROWS consecutive rows j of one token, over every slot and every 2048-column segment of F:
// the (slot, segment) units are dealt out to its wavefronts.  A wavefront keeps the activations of its unit in
// registers, streams the unit's piece of every row and adds gate * partial into per-lane, per-row accumulators;
// only after its last unit are the accumulators summed over the lanes (once per row instead of once per row and
// segment), then over the wavefronts through LDS in a fixed order, and y is written: no partial sums in memory
// and no separate combining launch.
// What is not streaming is start-up: until the first rows are requested the memory stands idle (a launch of 17 us over eight
// stacked layers, of 5 over small experts, waited 1.5 us for pair, expert, bit width and table entry, one after the other).  So
// the pair's entry comes ready from the first phase, in one scalar load for both of a round's units; the activations are
// requested with the first two batches of rows and not ahead of them; and the code in front of the loads is short.  From the
// kernel's start to the first requests 1.5 -> 0.5 us; one token, us a step before / after: eight of 128 experts 2048 x 768, 4/2
// bits 23.5 / 22.0, 4096 x 14336 16/4/2 bits 80.7 / 78.4, six of 64 1024 x 3072 31.1 / 29.9; 21 shapes 0.97.

// rows a wavefront requests at a time: two batches at least
template <int BITS, int ROWS> struct Phase2Rows { static constexpr int R = (ROWS == 4) ? 2 : (BITS == 16 || BITS == 8 || ROWS == 8) ? 4 : 8; };

constexpr int kP2MaxWaves = 8;

// fp32 intermediate against bf16 weights
struct LaneH {
    float v[4][8];
};

template <int NCH>
__device__ __forceinline__ float dot_row_h(const RowRegs<16, 1>& rr, const LaneH& lh)
{
    float acc = 0.0f;
#pragma unroll
    for (int c = 0; c < NCH; c++) {
        const uint4 u = rr.c[0][c];
        acc = fmaf(bf16_lo(u.x), lh.v[c][0], acc); acc = fmaf(bf16_hi(u.x), lh.v[c][1], acc);
        acc = fmaf(bf16_lo(u.y), lh.v[c][2], acc); acc = fmaf(bf16_hi(u.y), lh.v[c][3], acc);
        acc = fmaf(bf16_lo(u.z), lh.v[c][4], acc); acc = fmaf(bf16_hi(u.z), lh.v[c][5], acc);
        acc = fmaf(bf16_lo(u.w), lh.v[c][6], acc); acc = fmaf(bf16_hi(u.w), lh.v[c][7], acc);
    }
    return acc;
}

// one unit: segment `seg` of rows j_begin .. j_begin + ROWS - 1 (clamped to the last row H - 1).  arrange() makes the
// unit's activations of what was requested before: the first rows are on their way when it waits for them.
template <int BITS, int ROWS, int NCH, typename ArrangeFn, typename DotFn>
__device__ __forceinline__ void phase2_unit(const ExpertMat& m2, int F, int seg, int j_begin, int H,
                                            float gate, float (&tot)[ROWS], ArrangeFn arrange, DotFn dot)
{
    constexpr int R = Phase2Rows<BITS, ROWS>::R;
    constexpr int NB = ROWS / R;                 // 4 or 2 batches of rows
    static_assert(NB % 2 == 0, "batches come in pairs");
    const int lane = threadIdx.x & (kWave - 1);
    RowRegs<BITS, 1> ra[R], rb[R];                  // used in turn, as in phase 1
    auto fetch = [&](RowRegs<BITS, 1>(&dst)[R], int j0) {
#pragma unroll
        for (int i = 0; i < R; i++) load_row<BITS, 1, NCH>(m2, min(j0 + i, H - 1), F, seg, lane, dst[i]);
    };
    fetch(ra, j_begin);
    fetch(rb, j_begin + R);
    __builtin_amdgcn_sched_barrier(0);
    const auto lx = arrange();
#pragma unroll
    for (int bt = 0; bt < NB; bt += 2) {
#pragma unroll
        for (int i = 0; i < R; i++) tot[bt * R + i] = fmaf(gate, dot(ra[i], lx), tot[bt * R + i]);
        if (bt + 2 < NB) fetch(ra, j_begin + (bt + 2) * R);
#pragma unroll
        for (int i = 0; i < R; i++) tot[(bt + 1) * R + i] = fmaf(gate, dot(rb[i], lx), tot[(bt + 1) * R + i]);
        if (bt + 3 < NB) fetch(rb, j_begin + (bt + 3) * R);
    }
}

// Two units of narrow formats (int4, int2) side by side: a wavefront's start-up chain (pair -> activations and first rows) is
// a string of dependent latencies, and with 16 rows of int4 or int2 there is little streaming to hide the second unit's chain
// behind.  Taken together, both chains run at once.
template <int BA, int BB, int ROWS, typename ArrangeFn>
__device__ __forceinline__ void phase2_two_units(const ExpertMat& ma, const ExpertMat& mb, int F, int sa, int sb,
                                                 int j_begin, int H, float ga, float gb,
                                                 float (&tot)[ROWS], ArrangeFn arrange)
{
    constexpr int R = (ROWS == 4) ? 2 : 4;      // (eight int2 rows of both at a time spill: eight of 8 experts, 4096 x 6144, 97 / 87 us)
    constexpr int NB = ROWS / R;
    static_assert(NB % 2 == 0, "batches come in pairs");
    const int lane = threadIdx.x & (kWave - 1);
    RowRegs<BA, 1> a0[R], a1[R];
    RowRegs<BB, 1> b0[R], b1[R];
    auto fetch = [&](RowRegs<BA, 1>(&da)[R], RowRegs<BB, 1>(&db)[R], int j0) {
#pragma unroll
        for (int i = 0; i < R; i++) {
            const int row = min(j0 + i, H - 1);
            load_row<BA, 1>(ma, row, F, sa, lane, da[i]);
            load_row<BB, 1>(mb, row, F, sb, lane, db[i]);
        }
    };
    LaneX la[1], lb[1];
    auto finish = [&](const RowRegs<BA, 1>(&da)[R], const RowRegs<BB, 1>(&db)[R], int bt) {
#pragma unroll
        for (int i = 0; i < R; i++) {
            float acc = fmaf(ga, dot_row_q<BA, 1>(da[i], la), tot[bt * R + i]);
            tot[bt * R + i] = fmaf(gb, dot_row_q<BB, 1>(db[i], lb), acc);
        }
    };
    fetch(a0, b0, j_begin);
    __builtin_amdgcn_sched_barrier(0);
    arrange(la[0], lb[0]);
#pragma unroll
    for (int bt = 0; bt < NB; bt += 2) {
        fetch(a1, b1, j_begin + (bt + 1) * R);
        finish(a0, b0, bt);
        if (bt + 2 < NB) fetch(a0, b0, j_begin + (bt + 2) * R);
        finish(a1, b1, bt + 1);
    }
}

template <int ROWS, int NCH>
__global__ __launch_bounds__(kP2MaxWaves * kWave) void gemv_phase2_kernel(
    const float* __restrict__ hbuf, const PairDown* __restrict__ down, int H, int F, int k, int nseg, unsigned nseg_inv,
    int nwaves, int rounds, int out_dtype, void* __restrict__ y)
{
    __shared__ float s_red[kP2MaxWaves][ROWS];
    const int t = blockIdx.y;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    float tot[ROWS];
#pragma unroll
    for (int i = 0; i < ROWS; i++) tot[i] = 0.0f;
    const int units = k * nseg;
    // odd wavefronts take their units in reverse: the slots of a token differ in format (the later, the narrower),
    // and a compute unit should at any time hold wavefronts on wide, bandwidth-bound rows beside wavefronts on
    // narrow, instruction-bound ones instead of all of them on the same kind
    struct Unit {
        int p, s, b;
        float gate;
        ExpertMat m2;
    };
    auto unit_of = [&](int r) {
        const int u = wave + nwaves * ((wave & 1) ? rounds - 1 - r : r);
        const bool one = r < rounds && u < units;
        const int v = one ? u : 0;
        int slot = nseg == 1 ? v : (int)__umulhi((unsigned)v, nseg_inv);      // v / nseg, or one more
        if (slot * nseg > v) slot--;
        Unit un;
        un.s = v - slot * nseg;
        un.p = t * k + slot;
        const PairDown d = down[un.p];
        un.b = one ? d.bits : 0;
        un.gate = d.gate;
        un.m2.w = (const uint16_t*)d.codes;
        un.m2.q = (const uint8_t*)d.codes;
        un.m2.s = d.s;
        un.m2.z = d.z;
        return un;
    };
    // the unit's activations, of the lane's 32 columns in the order of quantised rows or in that of bf16 rows.  Columns past
    // the end are read as the row's first and made zero when the activations are used: a load under a condition, or anything
    // done to what it brought, would be waited for ahead of the first rows' loads.
    auto quant_x = [&](const Unit& un, float (&v)[32]) {
        const int col0 = un.s * kSeg + 32 * lane;
        const float* from = hbuf + (long)un.p * F + (col0 < F ? col0 : 0);
#pragma unroll
        for (int c = 0; c < 8; c++) {
            const float4 q = *reinterpret_cast<const float4*>(from + 4 * c);
            v[4 * c + 0] = q.x; v[4 * c + 1] = q.y; v[4 * c + 2] = q.z; v[4 * c + 3] = q.w;
        }
    };
    auto quant_end = [&](const Unit& un, float (&v)[32]) {
        const bool in = un.s * kSeg + 32 * lane < F;
#pragma unroll
        for (int i = 0; i < 32; i++) v[i] = in ? v[i] : 0.0f;
    };
    auto bf16_x = [&](const Unit& un, LaneH& lh) {
        const float* hrow = hbuf + (long)un.p * F;
#pragma unroll
        for (int c = 0; c < NCH; c++) {
            const int col = un.s * kSeg + (c * kWave + lane) * 8;
            const float* from = hrow + (col < F ? col : 0);
            const float4 lo = *reinterpret_cast<const float4*>(from);
            const float4 hi = *reinterpret_cast<const float4*>(from + 4);
            lh.v[c][0] = lo.x; lh.v[c][1] = lo.y; lh.v[c][2] = lo.z; lh.v[c][3] = lo.w;
            lh.v[c][4] = hi.x; lh.v[c][5] = hi.y; lh.v[c][6] = hi.z; lh.v[c][7] = hi.w;
        }
    };
    auto bf16_end = [&](const Unit& un, LaneH& lh) {
#pragma unroll
        for (int c = 0; c < NCH; c++) {
            const bool in = un.s * kSeg + (c * kWave + lane) * 8 < F;
#pragma unroll
            for (int i = 0; i < 8; i++) lh.v[c][i] = in ? lh.v[c][i] : 0.0f;
        }
    };
    for (int r = 0; r < rounds; r += 2) {
        const Unit ua = unit_of(r), ub = unit_of(r + 1);
        // (hidden from the compiler, which otherwise computes the addresses of every row in every format before the loop:
        // some two hundred instructions and spilled registers ahead of the first load)
        int j_begin = (int)blockIdx.x * ROWS;
        asm volatile("" : "+s"(j_begin));
        auto one_unit = [&](const Unit& un) {
            auto quantised = [&](auto bits) {
                constexpr int BITS = decltype(bits)::value;
                float v[32];
                quant_x(un, v);
                struct One {
                    LaneX l[1];
                };
                phase2_unit<BITS, ROWS, 4>(un.m2, F, un.s, j_begin, H, un.gate, tot, [&] {
                    One o;
                    quant_end(un, v);
                    arrange_lane_x<BITS>(v, o.l[0]);
                    return o;
                }, [](const RowRegs<BITS, 1>& rr, const One& o) { return dot_row_q<BITS, 1>(rr, o.l); });
            };
            if (un.b == 16) {
                LaneH lh;
                bf16_x(un, lh);
                phase2_unit<16, ROWS, NCH>(un.m2, F, un.s, j_begin, H, un.gate, tot, [&] {
                    bf16_end(un, lh);
                    return lh;
                },
                                           [](const RowRegs<16, 1>& rr, const LaneH& l) { return dot_row_h<NCH>(rr, l); });
            } else if (un.b == 8) {
                quantised(std::integral_constant<int, 8>());
            } else if (un.b == 4) {
                quantised(std::integral_constant<int, 4>());
            } else if (un.b == 2) {
                quantised(std::integral_constant<int, 2>());
            }
        };
        if ((ua.b == 4 || ua.b == 2) && (ub.b == 4 || ub.b == 2)) {
            auto both = [&](auto bits_a, auto bits_b) {
                constexpr int BA = decltype(bits_a)::value, BB = decltype(bits_b)::value;
                float va[32], vb[32];
                quant_x(ua, va);
                quant_x(ub, vb);
                phase2_two_units<BA, BB, ROWS>(ua.m2, ub.m2, F, ua.s, ub.s, j_begin, H, ua.gate, ub.gate, tot,
                                               [&](LaneX& la, LaneX& lb) {
                    quant_end(ua, va);
                    quant_end(ub, vb);
                    arrange_lane_x<BA>(va, la);
                    arrange_lane_x<BB>(vb, lb);
                });
            };
            const std::integral_constant<int, 4> four;
            const std::integral_constant<int, 2> two;
            if (ua.b == 4 && ub.b == 4) both(four, four);
            else if (ua.b == 4) both(four, two);
            else if (ub.b == 4) both(two, four);
            else both(two, two);
        } else {
            one_unit(ua);
            one_unit(ub);
        }
    }
    // lanes, then wavefronts (in wavefront order: the result does not depend on timing)
    float o = 0.0f;
#pragma unroll
    for (int i = 0; i < ROWS; i++) {
        const float r = wave_sum_dpp(tot[i]);
        if (lane == i) o = r;
    }
    if (lane < ROWS) s_red[wave][lane] = o;
    __syncthreads();
    const int j = (int)blockIdx.x * ROWS + (int)threadIdx.x;
    if (threadIdx.x < ROWS && j < H) {
        float acc = 0.0f;
        for (int wv = 0; wv < nwaves; wv++) acc += s_red[wv][threadIdx.x];
        const long i = (long)t * H + j;
        if (out_dtype == DYMOE_OUT_F32) reinterpret_cast<float*>(y)[i] = acc;
        else reinterpret_cast<uint16_t*>(y)[i] = (uint16_t)f32_to_bf16_bits(acc);
    }
}

// rows per workgroup of the first phase: 64 on the Mixtral-shaped decode layer (measured: beat 16..128), which makes 448
// workgroups; smaller layers get fewer rows per workgroup so that the launch still fills the chip
static int phase1_rows_per_block(long rows_total)
{
    int r = 64;
    while (r > 8 && rows_total / r < 384) r >>= 1;
    return r;
}

static int phase2_launch(dymoe_ctx* ctx, const float* hbuf, const PairDown* down, int T, int H, int F, int k, int out_dtype,
                         void* y, hipStream_t st)
{
    // as many wavefronts as (slot, segment) units, at most kP2MaxWaves; of the counts that need the
    // fewest rounds the smallest, so that no wavefront idles through the last round
    const int nseg2 = (F + kSeg - 1) / kSeg;
    const int units = k * nseg2;
    int nwaves = units < kP2MaxWaves ? units : kP2MaxWaves;
    const int rounds = (units + nwaves - 1) / nwaves;
    while (nwaves > 1 && (units + nwaves - 2) / (nwaves - 1) == rounds) nwaves--;
    const unsigned nseg_inv = (unsigned)((1ull << 32) / (unsigned)nseg2 + 1);      // (one segment: the kernel does not ask)
    // 16 rows per workgroup, fewer while the workgroups then still find a compute unit each: more of them on a unit only
    // repeat the start-up chain.  One token, us with 16 / 8 / 4 rows: H = 4096, F = 14336, int4 18 / 23 / -; 2048 x 768, eight
    // experts 8.9 / 7.0 / 8.5; 1024 x 3072 9.2 / 7.0 / 5.7; 512 x 1024 8.5 / 6.3 / 5.0; two tokens of 2048 x 768 12.3 / 14.6 / 18.6.
    int rows = 16;
    while (rows > 4 && (long)T * ((H + rows / 2 - 1) / (rows / 2)) <= ctx->num_cu) rows /= 2;
    const dim3 g2((unsigned)((H + rows - 1) / rows), (unsigned)T), block((unsigned)(nwaves * kWave));
    auto go = [&](auto kernel) {
        dymoe_launch(ctx, DYMOE_K_GEMV_PHASE2, kernel, g2, block, 0, st, hbuf, down, H, F, k, nseg2, nseg_inv, nwaves, rounds,
                     out_dtype, y);
    };
    // a segment's bf16 rows are four chunks of 512 columns: rows of at most 1024 columns need no more than two (2048 x 768,
    // eight bf16 experts: 12.4 us with all four, lanes past the end re-reading the tail, 10.2 with two)
    if (F <= kSeg / 2) rows == 4 ? go(gemv_phase2_kernel<4, 2>) : rows == 8 ? go(gemv_phase2_kernel<8, 2>) : go(gemv_phase2_kernel<16, 2>);
    else rows == 4 ? go(gemv_phase2_kernel<4, 4>) : rows == 8 ? go(gemv_phase2_kernel<8, 4>) : go(gemv_phase2_kernel<16, 4>);
    DYMOE_HIP_LAUNCH_CHECK();
    return DYMOE_OK;
}

int ffn_gemv_launch(dymoe_ctx* ctx, const void* x, const int32_t* idx, const float* w,
                    const uint8_t* bits, const dymoe_expert_fmt* table, int T, int H, int F, int E,
                    int k, int out_dtype, void* y, void* workspace, hipStream_t st)
{
    const FfnLayout L = ffn_layout(T, H, F, E, k);
    float* hbuf = reinterpret_cast<float*>((char*)workspace + L.hbuf);
    PairDown* down = reinterpret_cast<PairDown*>((char*)workspace + L.part);    // room for 4 H bytes a pair, H >= 64
    const int P = T * k;
    const int nseg1 = (H + kSeg - 1) / kSeg;
    const int rows1 = phase1_rows_per_block((long)F * P);
    const dim3 g1((unsigned)((F + rows1 - 1) / rows1), (unsigned)P);
    const uint16_t* xb = (const uint16_t*)x;
    {
        switch (nseg1) {
        case 1: dymoe_launch(ctx, DYMOE_K_GEMV_PHASE1, (gemv_phase1_kernel<1>), g1, dim3(kGvThreads), 0, st, xb, idx, w, bits, table, H, F, E, k, rows1, hbuf, down, ctx->device_flags); break;
        case 2: dymoe_launch(ctx, DYMOE_K_GEMV_PHASE1, (gemv_phase1_kernel<2>), g1, dim3(kGvThreads), 0, st, xb, idx, w, bits, table, H, F, E, k, rows1, hbuf, down, ctx->device_flags); break;
        case 3: dymoe_launch(ctx, DYMOE_K_GEMV_PHASE1, (gemv_phase1_kernel<3>), g1, dim3(kGvThreads), 0, st, xb, idx, w, bits, table, H, F, E, k, rows1, hbuf, down, ctx->device_flags); break;
        case 4: dymoe_launch(ctx, DYMOE_K_GEMV_PHASE1, (gemv_phase1_kernel<4>), g1, dim3(kGvThreads), 0, st, xb, idx, w, bits, table, H, F, E, k, rows1, hbuf, down, ctx->device_flags); break;
        default: return DYMOE_ENOTSUP;
        }
    }
    DYMOE_HIP_LAUNCH_CHECK();
    return phase2_launch(ctx, hbuf, down, T, H, F, k, out_dtype, y, st);
}

// Whether the fused decode step covers these sizes.
bool decode_fused_fits(int T, int H, int E, int k)
{
    return T >= 1 && T <= kFusedMaxTokens && E <= 64 && k <= kFusedMaxK && H % 64 == 0 && H <= 4 * kSeg;
}

// The logits of a launch of their own wait in the workspace's part area, P * H floats at least.
static bool logits_have_room(int H, int E, int k) { return (size_t)E <= (size_t)k * H; }

// Where the logits come from: a launch of their own (3 us) unless a workgroup has all the router rows it needs in one trip to
// memory (4 wavefronts, two rows each up to 4096 columns): every further trip costs every workgroup of the first phase 2 to 3
// us.  us a step, in the workgroups / apart: 8 experts x 4096, one token 15.2 / 16.5, four 32.0 / 30.8; 16 x 4096 20.5 / 19.4;
// 30 x 2048 18.3 / 15.4; 60 x 512 21.7 / 14.0; 64 x 1024, four tokens 71.9 / 38.5.
// With no more workgroups than compute units, nothing waits for a workgroup's trips but itself: two trips then cost what the launch
// does (and the host a launch less, which is what small layers called one by one wait for: 2 tokens x 8 experts, 256 x 128, 13.8 /
// 16.8 us a call), and from 2049 columns on the launch of few workgroups that makes the logits is no faster than a trip per token (two
// for rows of 6144 columns on).  In / apart, up to a workgroup per compute unit: 2 tokens x 4 experts x 8192 21.4 / 23.9, 4 x 2
// 26.5 / 31.4, 1 x 8 x 6144 20.2 / 20.9, 2 x 6 x 4096 18.5 / 19.2; but 1 x 9 x 6144 the same, 2 x 6 x 4160 the same, 4 x 6 x 4160 -1.5,
// 2 x 10 x 4096 -1.5, 4 x 4 x 2048 -1.4; above: 4 x 2 x 8192 -1.2, 2 x 4 x 6144 -2.2, 1 x 8 x 4160 -2.7.
static bool fused_logits_apart(const dymoe_ctx* ctx, int T, int H, int F, int E, int k)
{
    const int trip = H <= 2 * kSeg ? 2 * kGvWaves : kGvWaves;
    if (!logits_have_room(H, E, k) || (long)T * E <= trip) return false;
    const int rows = phase1_rows_per_block((long)F * T * k);
    const long workgroups = (long)((F + rows - 1) / rows) * T * k;
    if (workgroups > ctx->num_cu) return true;
    const int trips = (E + trip - 1) / trip;
    return !(T * trips <= 2 || (H > kSeg && (trips == 1 || (trips == 2 && H >= 3 * kSeg))));
}

// ... and the decode layer: up to kFusedMaxE experts, and one token behind the layer before's residual
bool decode_layer_fits(int T, int H, int E, int k, bool residual)
{
    if (T < 1 || T > (residual ? 1 : kFusedMaxTokens) || E > kFusedMaxE || k > kFusedMaxK || H % 64 != 0 || H > 4 * kSeg) return false;
    return E <= 64 || logits_have_room(H, E, k);
}

int front_logits_launch(dymoe_ctx* ctx, const void* x, const float* y_prev, float alpha, void* h_out, const void* wg, const float* bias,
                        int T, int H, int E, float* logits, hipStream_t st);
int front_finish_launch(dymoe_ctx* ctx, int T, int E, int k, int renorm, int32_t* idx, float* w, float* probs, const TierTable& tt,
                        int floor_bits, float* importance, int32_t* load, uint8_t* bits, int32_t* rank, hipStream_t st);

// y_prev not NULL: x is the layer before's input, y_prev its output, and the normalised row goes to h_out as well
int decode_fused_launch(dymoe_ctx* ctx, const void* x, const float* y_prev, float alpha, void* h_out, const void* wg, const float* bias,
                        const TierTable& tt, int floor_bits, const dymoe_expert_fmt* table, int T, int H, int F, int E, int k, int renorm,
                        int out_dtype, int32_t* idx, float* w, float* probs, float* importance, int32_t* load,
                        uint8_t* bits, int32_t* rank, void* y, void* workspace, hipStream_t st)
{
    const FfnLayout L = ffn_layout(T, H, F, E, k);
    float* hbuf = reinterpret_cast<float*>((char*)workspace + L.hbuf);
    // (not in the part area, whose logits the first phase still reads; 6 H bytes a token and up to kFusedMaxK pairs, H >= 64)
    static_assert(kFusedMaxK * sizeof(PairDown) <= 6 * 64, "the pairs' entries fit beside the logits");
    PairDown* down = reinterpret_cast<PairDown*>((char*)workspace + L.xh);
    const int P = T * k;
    const int nseg1 = (H + kSeg - 1) / kSeg;
    const int rows1 = phase1_rows_per_block((long)F * P);
    const dim3 g1((unsigned)((F + rows1 - 1) / rows1), (unsigned)P);
    FusedFront f = {};
    f.x = (const uint16_t*)x; f.y_prev = y_prev; f.alpha = alpha; f.h_out = (uint16_t*)h_out;
    f.wg = (const uint16_t*)wg; f.bias = bias; f.renorm = renorm; f.floor_bits = floor_bits; f.tiers = tt;
    f.idx = idx; f.w = w; f.probs = probs; f.importance = importance; f.load = load; f.bits = bits; f.rank = rank;
    // From 65 experts on the front end's outputs are a workgroup's work: ranking them and writing everything down is 5 us on top of
    // what each does for itself, and the workgroup that went on to rows after it was the last to end.  With a workgroup of its own,
    // where that is resident beside the others (one token, us a step, without / with: eight of 128 experts, 2048 x 768, int4 20.6 /
    // 18.1, bf16 24.1 / 23.6; four tokens, 1024 x 768, 36.2 / 35.1); up to 64 experts it is 0.6 us and not the last.
    // Resident together: four, two or one per compute unit by the registers of 1, 2 or more segments.
    const long resident = (nseg1 == 1 ? 4L : nseg1 == 2 ? 2L : 1L) * ctx->num_cu;
    const long workgroups = (long)g1.x * g1.y;
    const bool front_apart = E > 64 && workgroups + 1 <= resident;
    const dim3 grid = front_apart ? dim3((unsigned)workgroups + 1) : g1;
    auto go = [&](auto kernel) {
        dymoe_launch(ctx, DYMOE_K_GEMV_PHASE1, kernel, grid, dim3(kGvThreads), 0, st, f, table, T, H, F, E, k,
                     (int)front_apart, rows1, hbuf,
                     down, ctx->device_flags);
    };
    // NCH: 16-byte chunks of an activation row per lane, as in dymoe_decode_front (8 up to 4096 columns, then 16)
    auto by_width = [&](auto experts, auto front) {
        constexpr int NC = decltype(experts)::value, FR = decltype(front)::value;
        switch (nseg1) {
        case 1: go(decode_fused_phase1_kernel<1, 8, NC, FR>); break;
        case 2: go(decode_fused_phase1_kernel<2, 8, NC, FR>); break;
        case 3: go(decode_fused_phase1_kernel<3, 16, NC, FR>); break;
        default: go(decode_fused_phase1_kernel<4, 16, NC, FR>); break;
        }
    };
    if (nseg1 > 4) return DYMOE_ENOTSUP;
    if (fused_logits_apart(ctx, T, H, F, E, k)) {
        // More workgroups than are resident together would do softmax, top-k and ranking once per round: then a launch does them, and the first phase is the stand-alone one.
        // us a step, in every round / once: 4 tokens x 8 of 100 experts, 7360 x 192 (768 workgroups) 121 / 112, 4 x 8 of 8, 4096 x
        // 4096 (2048) 236 / 208, 2 x 8 of 65, 6016 x 192 (384) 4.8 more; up to one round 2 to 4 less (4 x 8 of 128, 4096 x 192 (384)
        // 3.3, 2048 x 768 (768) 3.6).
        const bool once = workgroups > resident;
        float* logits = (once && probs) ? probs : reinterpret_cast<float*>((char*)workspace + L.part);
        int rc = front_logits_launch(ctx, x, y_prev, alpha, h_out, wg, bias, T, H, E, logits, st);
        if (rc != DYMOE_OK) return rc;
        if (y_prev) f.x = (const uint16_t*)h_out;
        if (once) {
            rc = front_finish_launch(ctx, T, E, k, renorm, idx, w, logits, tt, floor_bits, importance, load, bits, rank, st);
            if (rc != DYMOE_OK) return rc;
            return ffn_gemv_launch(ctx, f.x, idx, w, bits, table, T, H, F, E, k, out_dtype, y, workspace, st);
        }
        f.logits = logits;
        if (E <= 64) by_width(std::integral_constant<int, 1>(), std::integral_constant<int, kFrontLogits>());
        else by_width(std::integral_constant<int, 2>(), std::integral_constant<int, kFrontLogits>());
    } else if (y_prev) {
        by_width(std::integral_constant<int, 1>(), std::integral_constant<int, kFrontResidual>());
    } else {
        by_width(std::integral_constant<int, 1>(), std::integral_constant<int, kFrontRouter>());
    }
    DYMOE_HIP_LAUNCH_CHECK();
    return phase2_launch(ctx, hbuf, down, T, H, F, k, out_dtype, y, st);
}

}  // namespace dymoe
