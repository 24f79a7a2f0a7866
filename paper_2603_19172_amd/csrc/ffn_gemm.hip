// Prefill path of the mixed-precision SwiGLU expert FFN: tokens grouped by
// expert, one MFMA grouped GEMM per projection, all experts in one launch.
//
// Work unit: up to 128 token rows of one expert x (4 wavefronts x 2 strips of
// 32 weight rows), K walked in tiles of 128.
//  * Weights never touch LDS.  They are stored in 32 x 128 tiles whose byte
//    order is the MFMA A-operand order (lane (r, kb) owns row r, columns
//    64 kb .. 64 kb + 64, one quantisation group), so every load instruction of
//    a wavefront reads 1 KiB of contiguous memory straight into the registers
//    the MFMA consumes (bf16) or the dequantiser consumes (int4 / int2).
//  * The token tile is shared by the 4 wavefronts through a double-buffered
//    LDS tile; it is copied from a 16-bit copy of the activations that is
//    already in the column order the code fields come out of a dword, so
//    staging is a plain copy: global memory -> LDS directly
//    (global_load_lds_dwordx4), stored swizzled so that the operand reads are
//    free of bank conflicts without padding.
//  * bf16 experts: v_mfma_f32_32x32x16_bf16 on the bf16 activations.
//    int4 / int2 experts: v_mfma_f32_32x32x16_f16 on an fp16 copy of the
//    activations; weights become fp16 in registers: a code field OR-ed into the
//    mantissa of 2^n (n such that the field's lowest bit weighs one) is the
//    number 2^n + q; subtracting 2^n is exact; then one packed fma(q, s, m).
//  * A workgroup is four wavefronts, one per SIMD, and two workgroups share a
//    compute unit: the two wavefronts of a SIMD belong to different workgroups,
//    so one's barrier, waits, prologue and epilogue are covered by the other's
//    MFMA work.
//  * Calls of few tokens per expert plan tiles of 32 rows and take gemm_small_kernel, which keeps both operands in registers.
//  * Results leave through LDS: in the MFMA result layout a lane holds a few
//    outputs of one token's row, so stores made from it would touch 32 rows per
//    instruction; the token-tile buffers, free after the K loop, turn the
//    rows round so that 16 lanes store 256 contiguous bytes of one row.
#include <math.h>

#include "common.hpp"
#include "ffn_layout.hpp"
#include "plan_device.hpp"

namespace dymoe {

constexpr int kGmThreads = 256;
constexpr int kGmWaves = 4;         // one per SIMD; two workgroups share a compute unit
constexpr int kBK = 128;            // K-tile
constexpr int kXsBufBytes = kGemmTileTall * kBK * 2;   // one token tile in LDS: up to 160 rows x 256 bytes, no padding

// ----------------------------------------------------------------------------
// weight strips (32 rows x one K-tile of 128), as one lane holds them

template <int BITS> struct StripRaw;
template <> struct StripRaw<16> { uint4 r[8]; };
template <> struct StripRaw<8> { uint4 r[4]; uint32_t s2, m2; };
template <> struct StripRaw<4> { uint4 r[2]; uint32_t s2, m2; };
template <> struct StripRaw<2> { uint4 r[1]; uint32_t s2, m2; };

struct MatPtr {
    const uint16_t* w;    // bf16 row-major
    const char* wt;       // bf16 tiles (may be null)
    const char* q;        // packed codes, tile layout
    const uint16_t* s;    // fp16 scale, tile layout
    const uint16_t* z;    // fp16 zero, tile layout
};

__device__ __forceinline__ MatPtr mat_ptr(const dymoe_expert_fmt& ex, int mat, int b)
{
    MatPtr m;
    m.w = reinterpret_cast<const uint16_t*>(ex.w[mat]);
    m.wt = reinterpret_cast<const char*>(ex.wt[mat]);
    m.q = reinterpret_cast<const char*>((b == 8) ? ex.q8[mat] : (b == 4) ? ex.q4[mat] : ex.q2[mat]);
    m.s = reinterpret_cast<const uint16_t*>((b == 8) ? ex.s8[mat] : (b == 4) ? ex.s4[mat] : ex.s2[mat]);
    m.z = reinterpret_cast<const uint16_t*>((b == 8) ? ex.z8[mat] : (b == 4) ? ex.z4[mat] : ex.z2[mat]);
    return m;
}

__device__ __forceinline__ uint32_t deq_pair(uint32_t biased, uint32_t bias2, uint32_t s2, uint32_t m2)
{
    const half2_t q = __builtin_bit_cast(half2_t, biased) - __builtin_bit_cast(half2_t, bias2);  // exact
    const half2_t r = __builtin_elementwise_fma(q, __builtin_bit_cast(half2_t, s2),
                                                __builtin_bit_cast(half2_t, m2));
    return __builtin_bit_cast(uint32_t, r);
}

// A fragments of MFMA sub-steps 2*jj and 2*jj+1 (8 k each) of one strip
template <int BITS>
__device__ __forceinline__ void strip_frags(const StripRaw<BITS>& raw, int jj, uint4& f0, uint4& f1)
{
    if constexpr (BITS == 16) {
        f0 = raw.r[2 * jj];
        f1 = raw.r[2 * jj + 1];
    } else if constexpr (BITS == 8) {
        // 16 codes, one per byte, in k order: a byte b becomes the fp16 number 1024 + b
        const uint4 q = raw.r[jj];
        f0.x = deq_pair(__builtin_amdgcn_perm(0x64646464u, q.x, 0x04010400u), 0x64006400u, raw.s2, raw.m2);
        f0.y = deq_pair(__builtin_amdgcn_perm(0x64646464u, q.x, 0x04030402u), 0x64006400u, raw.s2, raw.m2);
        f0.z = deq_pair(__builtin_amdgcn_perm(0x64646464u, q.y, 0x04010400u), 0x64006400u, raw.s2, raw.m2);
        f0.w = deq_pair(__builtin_amdgcn_perm(0x64646464u, q.y, 0x04030402u), 0x64006400u, raw.s2, raw.m2);
        f1.x = deq_pair(__builtin_amdgcn_perm(0x64646464u, q.z, 0x04010400u), 0x64006400u, raw.s2, raw.m2);
        f1.y = deq_pair(__builtin_amdgcn_perm(0x64646464u, q.z, 0x04030402u), 0x64006400u, raw.s2, raw.m2);
        f1.z = deq_pair(__builtin_amdgcn_perm(0x64646464u, q.w, 0x04010400u), 0x64006400u, raw.s2, raw.m2);
        f1.w = deq_pair(__builtin_amdgcn_perm(0x64646464u, q.w, 0x04030402u), 0x64006400u, raw.s2, raw.m2);
    } else if constexpr (BITS == 4) {
        const uint4 q = raw.r[jj >> 1];
        const uint32_t w0 = (jj & 1) ? q.z : q.x;
        const uint32_t w1 = (jj & 1) ? q.w : q.y;
        // k order inside a fragment: 0,4,1,5,2,6,3,7
        uint32_t v = w0, v8 = w0 >> 8;
        f0.x = deq_pair(and_or(v, 0x000F000Fu, 0x64006400u), 0x64006400u, raw.s2, raw.m2);
        f0.y = deq_pair(and_or(v, 0x00F000F0u, 0x54005400u), 0x54005400u, raw.s2, raw.m2);
        f0.z = deq_pair(and_or(v8, 0x000F000Fu, 0x64006400u), 0x64006400u, raw.s2, raw.m2);
        f0.w = deq_pair(and_or(v8, 0x00F000F0u, 0x54005400u), 0x54005400u, raw.s2, raw.m2);
        v = w1; v8 = w1 >> 8;
        f1.x = deq_pair(and_or(v, 0x000F000Fu, 0x64006400u), 0x64006400u, raw.s2, raw.m2);
        f1.y = deq_pair(and_or(v, 0x00F000F0u, 0x54005400u), 0x54005400u, raw.s2, raw.m2);
        f1.z = deq_pair(and_or(v8, 0x000F000Fu, 0x64006400u), 0x64006400u, raw.s2, raw.m2);
        f1.w = deq_pair(and_or(v8, 0x00F000F0u, 0x54005400u), 0x54005400u, raw.s2, raw.m2);
    } else {
        const uint4 q = raw.r[0];
        const uint32_t v = (jj == 0) ? q.x : (jj == 1) ? q.y : (jj == 2) ? q.z : q.w;
        const uint32_t v10 = v >> 10;
        // 16 codes of the dword; k order 0,8,1,9,2,10,3,11 | 4,12,5,13,6,14,7,15
        f0.x = deq_pair(and_or(v, 0x00030003u, 0x64006400u), 0x64006400u, raw.s2, raw.m2);
        f0.y = deq_pair(and_or(v, 0x000C000Cu, 0x5C005C00u), 0x5C005C00u, raw.s2, raw.m2);
        f0.z = deq_pair(and_or(v, 0x00300030u, 0x54005400u), 0x54005400u, raw.s2, raw.m2);
        f0.w = deq_pair(and_or(v, 0x00C000C0u, 0x4C004C00u), 0x4C004C00u, raw.s2, raw.m2);
        f1.x = deq_pair(and_or(v, 0x03000300u, 0x44004400u), 0x44004400u, raw.s2, raw.m2);
        f1.y = deq_pair(and_or(v10, 0x00030003u, 0x64006400u), 0x64006400u, raw.s2, raw.m2);
        f1.z = deq_pair(and_or(v10, 0x000C000Cu, 0x5C005C00u), 0x5C005C00u, raw.s2, raw.m2);
        f1.w = deq_pair(and_or(v10, 0x00300030u, 0x54005400u), 0x54005400u, raw.s2, raw.m2);
    }
}

template <int BITS>
__device__ __forceinline__ float16_t mfma16(const uint4 a, const uint4 b, const float16_t c)
{
    if constexpr (BITS == 16)
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a),
                                                      __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8_t, a),
                                                      __builtin_bit_cast(half8_t, b), c, 0, 0, 0);
}

// address of this lane's slice of the K-tiles of one 32-row strip
struct StripSrc {
    const char* p;        // this lane's first 16 bytes of K-tile 0 (bf16 tiles or rows, or packed codes)
    const uint16_t* s;    // scale / zero at this lane's slot of K-tile 0 (quantised only)
    const uint16_t* z;
    int kt_stride;        // bytes from one K-tile to the next
    int c_stride;         // bytes from one 16-byte chunk of the lane's slice to the next
};

template <int BITS>
__device__ __forceinline__ StripSrc strip_src(const MatPtr& m, long nt, int K, int lane)
{
    StripSrc src;
    const long tile_row = nt * (K >> 7);
    src.s = m.s + tile_row * 64 + (uint32_t)lane;
    src.z = m.z + tile_row * 64 + (uint32_t)lane;
    if constexpr (BITS == 16) {
        if (m.wt) {          // tiles: chunk c of every lane sits in one 1 KiB run
            src.p = m.wt + tile_row * 8192 + (uint32_t)(lane * 16);
            src.kt_stride = 8192;
            src.c_stride = 1024;
        } else {             // rows: the lane's 64 columns are contiguous
            src.p = reinterpret_cast<const char*>(m.w + (nt * 32 + (lane & 31)) * K + 64 * (lane >> 5));
            src.kt_stride = 256;
            src.c_stride = 16;
        }
    } else {
        src.p = m.q + tile_row * (512 * BITS) + (uint32_t)(lane * 16);      // 32 x 128 codes of BITS bits: 512 * BITS bytes per tile
        src.kt_stride = 512 * BITS;
        src.c_stride = 1024;
    }
    return src;
}

// chunk c of the lane's slice of K-tile kt: bf16 c = 0..7 (8 columns each),
// int8 c = 0..3 (16 codes each), int4 c = 0..1 (32 codes each), int2 c = 0 (64 codes)
template <int BITS>
__device__ __forceinline__ uint4 load_chunk(const StripSrc& src, int kt, int c)
{
    if constexpr (BITS == 16) return load_global<uint4>(src.p + (long)kt * src.kt_stride + c * src.c_stride);
    else if constexpr (BITS == 8) return load_global<uint4>(src.p + (long)kt * 4096 + c * 1024);
    else if constexpr (BITS == 4) return load_global<uint4>(src.p + (long)kt * 2048 + c * 1024);
    else return load_global<uint4>(src.p + (long)kt * 1024);
}

template <int BITS>
__device__ __forceinline__ void load_scale_zero(const StripSrc& src, int kt, StripRaw<BITS>& raw)
{
    if constexpr (BITS != 16) {
        // the 16-bit values as loaded; adopt_strip() duplicates them into both halves
        raw.s2 = load_global<uint16_t>(src.s + kt * 64);
        raw.m2 = load_global<uint16_t>(src.z + kt * 64);
    }
}

// Make a freshly loaded strip the current one.  Touching the loaded values is
// left to this point, a whole K-tile after the request, so nothing waits for a
// load right after issuing it.
template <int BITS>
__device__ __forceinline__ void adopt_strip(StripRaw<BITS>& cur, const StripRaw<BITS>& next)
{
    cur = next;
    if constexpr (BITS != 16) {
        cur.s2 |= cur.s2 << 16;
        cur.m2 |= cur.m2 << 16;
    }
}

template <int BITS>
__device__ __forceinline__ void load_strip(const StripSrc& src, int kt, StripRaw<BITS>& raw)
{
    constexpr int kChunks = (BITS == 16) ? 8 : (BITS == 8 ? 4 : (BITS == 4 ? 2 : 1));
#pragma unroll
    for (int c = 0; c < kChunks; c++) raw.r[c] = load_chunk<BITS>(src, kt, c);
    load_scale_zero<BITS>(src, kt, raw);
}

// 16 bytes of LDS at a byte address
__device__ __forceinline__ uint4 lds_read16(uint32_t addr)
{
    const u32x4_t v = *(const __attribute__((address_space(3))) u32x4_t*)(uintptr_t)addr;
    return __builtin_bit_cast(uint4, v);
}

__device__ __forceinline__ void lds_write16(uint32_t addr, const uint4 v)
{
    *(__attribute__((address_space(3))) u32x4_t*)(uintptr_t)addr = __builtin_bit_cast(u32x4_t, v);
}

typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ void lds_write8(uint32_t addr, const uint2 v)
{
    *(__attribute__((address_space(3))) u32x2_t*)(uintptr_t)addr = __builtin_bit_cast(u32x2_t, v);
}

__device__ __forceinline__ uint32_t lds_read4(uint32_t addr)
{
    return *(const __attribute__((address_space(3))) uint32_t*)(uintptr_t)addr;
}

__device__ __forceinline__ void lds_write4(uint32_t addr, uint32_t v)
{
    *(__attribute__((address_space(3))) uint32_t*)(uintptr_t)addr = v;
}

// second GEMM's epilogue: a wavefront's own LDS area, 32 rows of 256 bytes + 16 of padding
constexpr uint32_t kEpiRowBytes = 272;
constexpr uint32_t kEpiWaveBytes = 32 * kEpiRowBytes;
static_assert(kGmWaves * kEpiWaveBytes <= (uint32_t)kXsBufBytes, "the epilogue areas fit in the first token-tile buffer");
static_assert(kGemmTileTall * kEpiRowBytes <= 2 * (uint32_t)kXsBufBytes, "the first GEMM's output rows fit in the two buffers");

// The token operands of one MFMA step (two 16-byte chunks of one row).
struct XOps {
    uint4 t0, t1;
};

// Quarters JJ0 .. JJ1-1 of one K-tile of MFMAs for NTF token fragments (32 tokens each).
// A step is one (quarter, fragment) pair: four MFMAs on two LDS chunks.  The
// chunks of step s+1 are requested before the MFMAs of step s are issued, so the
// LDS latency hides behind arithmetic; the operands of a tile's first step come
// in through `ops`.  Scheduling barriers keep this order.
// bf16 (64 registers of raw weights per K-tile): the loads of the next K-tile
// are woven into the sequence; every weight register is refilled as soon as
// the last MFMA that reads it has been issued, so the next tile's weights are
// in flight during three quarters of this tile's arithmetic without a second
// set of registers.
// int8 (16 registers of codes per strip): refilled in place like bf16; only the
// scale and zero of the next tile wait in registers of their own.
// int4 / int2 (10 / 6 registers per strip): the next tile's codes were already
// requested into a second register set before this call; nothing to load here.
template <int BITS, int NTF, int JJ0, int JJ1>
__device__ __forceinline__ void compute_ktile(StripRaw<BITS>& ra, StripRaw<BITS>& rb,
                                              const StripSrc& sa, const StripSrc& sb, int kt_next,
                                              uint32_t xa, XOps& ops, float16_t (&acc)[2][NTF])
{
    constexpr int kStepMask = 0x2 | 0x4;            // VALU and SALU may cross; MFMA, LDS and global accesses may not
#pragma unroll
    for (int jj = JJ0; jj < JJ1; jj++) {
        uint4 a0, a1, b0, b1;
        strip_frags<BITS>(ra, jj, a0, a1);
        strip_frags<BITS>(rb, jj, b0, b1);
#pragma unroll
        for (int tf = 0; tf < NTF; tf++) {
            if constexpr (NTF == 5) {
                // five fragments: 160 accumulator registers leave no room for a second pair of operands, so a step
                // reads its own (the other wavefront of the SIMD covers the LDS latency)
                const uint32_t x0 = (xa ^ (uint32_t)(jj << 5)) + tf * (32 * kBK * 2);
                ops.t0 = lds_read16(x0);
                ops.t1 = lds_read16(x0 ^ 16u);
                __builtin_amdgcn_sched_barrier(kStepMask);
                acc[0][tf] = mfma16<BITS>(a0, ops.t0, acc[0][tf]);
                acc[1][tf] = mfma16<BITS>(b0, ops.t0, acc[1][tf]);
                acc[0][tf] = mfma16<BITS>(a1, ops.t1, acc[0][tf]);
                acc[1][tf] = mfma16<BITS>(b1, ops.t1, acc[1][tf]);
                __builtin_amdgcn_sched_barrier(kStepMask);
            } else {
            // next step: next fragment, else next quarter (nothing after the tile's last step)
            const bool wrap = (tf == NTF - 1);
            const bool last = wrap && jj == 3;
            const int njj = wrap ? jj + 1 : jj;
            const int ntf = wrap ? 0 : tf + 1;
            XOps nxt = ops;
            if (!last) {
                const uint32_t x0 = (xa ^ (uint32_t)(njj << 5)) + ntf * (32 * kBK * 2);
                nxt.t0 = lds_read16(x0);
                nxt.t1 = lds_read16(x0 ^ 16u);
            }
            __builtin_amdgcn_sched_barrier(kStepMask);
            acc[0][tf] = mfma16<BITS>(a0, ops.t0, acc[0][tf]);
            acc[1][tf] = mfma16<BITS>(b0, ops.t0, acc[1][tf]);
            acc[0][tf] = mfma16<BITS>(a1, ops.t1, acc[0][tf]);
            acc[1][tf] = mfma16<BITS>(b1, ops.t1, acc[1][tf]);
            ops = nxt;
            __builtin_amdgcn_sched_barrier(kStepMask);
            }
        }
        if constexpr (BITS == 16) {
            ra.r[2 * jj] = load_chunk<16>(sa, kt_next, 2 * jj);
            ra.r[2 * jj + 1] = load_chunk<16>(sa, kt_next, 2 * jj + 1);
            rb.r[2 * jj] = load_chunk<16>(sb, kt_next, 2 * jj);
            rb.r[2 * jj + 1] = load_chunk<16>(sb, kt_next, 2 * jj + 1);
            __builtin_amdgcn_sched_barrier(kStepMask);
        } else if constexpr (BITS == 8) {
            ra.r[jj] = load_chunk<8>(sa, kt_next, jj);
            rb.r[jj] = load_chunk<8>(sb, kt_next, jj);
            __builtin_amdgcn_sched_barrier(kStepMask);
        } else if constexpr (NTF == 5 && BITS == 4) {
            // five fragments: no second register set; each 16-byte chunk of codes serves two quarters and is
            // refilled when the second is done, half a tile before the next tile needs it
            if (jj & 1) {
                ra.r[jj >> 1] = load_chunk<4>(sa, kt_next, jj >> 1);
                rb.r[jj >> 1] = load_chunk<4>(sb, kt_next, jj >> 1);
                __builtin_amdgcn_sched_barrier(kStepMask);
            }
        }
    }
}

// Global-memory instructions issued per K-tile after the token-tile copies
// (every one of them unconditional): the copies are older than all of them, so
// "at most this many memory operations still in flight" means the copies landed.
template <int BITS>
constexpr int ktile_loads()
{
    return BITS == 16 ? 16 : (BITS == 8 ? 12 : (BITS == 4 ? 8 : 6));
}

// ----------------------------------------------------------------------------
// Token tile: global memory -> LDS without passing through registers.
//
// global_load_lds_dwordx4 writes the 16 bytes a lane fetched to
// LDS[M0 + 16 * lane]: one instruction fills 1 KiB = 4 tile rows of 256 bytes.
// The lane chooses WHAT it fetches, so the tile is stored swizzled for free:
// row r keeps its 16-byte chunk c at chunk position c ^ (r & 15).  The MFMA
// operand reads (lane = row, fixed c) then fall on 16 different chunk
// positions for 16 consecutive rows, i.e. on all banks once.
// Wavefront w fills rows 32 i + 4 w .. + 3 (i = 0 .. NTF-1); a thread's rows
// all have the same r & 15, hence the same source chunk.
constexpr int kRowsPerCopy = 4 * kGmWaves;      // tile rows the workgroup fills with one instruction per wavefront

template <int NTF>
struct XStage {
    static constexpr int kCopies = 32 * NTF / kRowsPerCopy;
    const char* base;            // start of the activation matrix (the same in every lane)
    uint32_t off[kCopies];       // byte offset of this thread's 16 bytes of K-tile 0 in each of its rows
    uint32_t lds;                // LDS address of lane 0's slot of the wavefront's first unit, buffer 0
};

template <int NTF>
__device__ __forceinline__ void copy_tile(const XStage<NTF>& st, int kt, int buf)
{
    const char* base = st.base + (long)kt * (kBK * 2);
#pragma unroll
    for (int i = 0; i < XStage<NTF>::kCopies; i++)
        lds_copy16(base, st.off[i], st.lds + buf * kXsBufBytes + i * (kRowsPerCopy * kBK * 2));
}

// ----------------------------------------------------------------------------
// MODE 1: h = silu(x W1^T) * (x W3^T)   strips = (W1 rows, W3 rows) of the same 32 features
// MODE 2: o = h W2^T                     strips = two adjacent groups of 32 rows of W2,
//                                        K-tiles [kt_begin, kt_end) of the split
template <int MODE, int BITS, int NTF>
__device__ __forceinline__ void gemm_tile(
    const uint16_t* __restrict__ act,   // MODE 1: [T,K] activations (gathered); MODE 2: [P,K] intermediate
    const int32_t* __restrict__ perm, int k_route, const dymoe_expert_fmt& ex, int K, int N,
    int kt_begin, int kt_end, int row0, int rows, int nblock, uint16_t* __restrict__ hout,
    float* __restrict__ oout, uint32_t xs_base)
{
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);     // (the same in every lane: addresses built from it stay scalar)
    const int ln = lane & 31;
    const int kb = lane >> 5;

    // strips of this wavefront (32-row tiles of the weight matrices)
    long nt_a, nt_b;
    MatPtr ma, mb;
    bool strip_ok[2];
    if (MODE == 1) {
        nt_a = nt_b = (long)nblock * kGmWaves + wave;
        ma = mat_ptr(ex, 0, BITS);
        mb = mat_ptr(ex, 1, BITS);
        strip_ok[0] = strip_ok[1] = nt_a * 32 < N;
    } else {
        nt_a = ((long)nblock * kGmWaves + wave) * 2;
        nt_b = nt_a + 1;
        ma = mb = mat_ptr(ex, 2, BITS);
        strip_ok[0] = nt_a * 32 < N;
        strip_ok[1] = nt_b * 32 < N;
    }
    if (!strip_ok[0]) nt_a = 0;   // idle strips stream tile row 0; their results are dropped
    if (!strip_ok[1]) nt_b = 0;

    float16_t acc[2][NTF];
#pragma unroll
    for (int s = 0; s < 2; s++)
#pragma unroll
        for (int tf = 0; tf < NTF; tf++)
#pragma unroll
            for (int i = 0; i < 16; i++) acc[s][tf][i] = 0.0f;

    // staging role: rows 16 i + 4 wave + lane / 16, physical chunk lane % 16.
    // Tile rows past the expert's last token re-read its last token: their
    // products are computed and dropped, and the loop stays branch-free.
    XStage<NTF> stage;
    {
        const int rb = 4 * wave + (lane >> 4);
        const int chunk = (lane & 15) ^ (rb & 15);
#pragma unroll
        for (int i = 0; i < XStage<NTF>::kCopies; i++) {
            const int r = min(kRowsPerCopy * i + rb, rows - 1);
            const long src_row = (MODE == 1) ? (long)(perm[row0 + r] / k_route) : (long)(row0 + r);
            stage.off[i] = (uint32_t)(src_row * K * 2 + 16 * chunk);     // < 4 GiB, checked by the launcher
        }
        stage.base = reinterpret_cast<const char*>(act);
        stage.lds = __builtin_amdgcn_readfirstlane(xs_base + wave * 1024);
    }
    // operand reads: lane (ln, kb) reads row 32 tf + ln, chunks 8 kb + 2 jj (+1)
    const uint32_t xa0 = xs_base + ln * (kBK * 2) + (((uint32_t)kb << 7) ^ ((uint32_t)(ln & 15) << 4));
    uint32_t xa = xa0;

    // K loop over two LDS buffers: the next token tile is copied into the other
    // buffer while this one is multiplied.  The two workgroups of a compute unit
    // run independently, so one's barrier, prologue and epilogue overlap the
    // other's arithmetic.
    const StripSrc sa = strip_src<BITS>(ma, nt_a, K, lane);
    const StripSrc sb = strip_src<BITS>(mb, nt_b, K, lane);
    StripRaw<BITS> ra, rb;
    copy_tile<NTF>(stage, kt_begin, 0);
    load_strip<BITS>(sa, kt_begin, ra);
    load_strip<BITS>(sb, kt_begin, rb);
    adopt_strip<BITS>(ra, ra);
    adopt_strip<BITS>(rb, rb);
    wait_lds_copies<0>();
    __syncthreads();
    int buf = 0;          // buffer of tile kt
    for (int kt = kt_begin; kt < kt_end; kt++) {
        // past the end the prefetches re-read the last tile instead of branching
        const int kn = min(kt + 1, kt_end - 1);
        copy_tile<NTF>(stage, kn, buf ^ 1);
        StripRaw<BITS> na, nb;
        constexpr bool kSecondSet = (BITS == 2) || (BITS == 4 && NTF != 5);    // next tile's codes in registers of their own
        if constexpr (kSecondSet) {
            load_strip<BITS>(sa, kn, na);
            load_strip<BITS>(sb, kn, nb);
            __builtin_amdgcn_sched_barrier(0);   // keep the requests up here, a whole tile ahead of their use
        }
        XOps ops;             // operands of the first step
        ops.t0 = lds_read16(xa);
        ops.t1 = lds_read16(xa ^ 16u);
        if constexpr (BITS == 8 || (BITS == 4 && NTF == 5)) {
            // the next tile's scale and zero are requested after the first quarter's
            // refills: a wait for a refilled register then never reaches back to
            // the copies issued at the top of the tile before a quarter has passed
            compute_ktile<BITS, NTF, 0, 1>(ra, rb, sa, sb, kn, xa, ops, acc);
            load_scale_zero<BITS>(sa, kn, na);
            load_scale_zero<BITS>(sb, kn, nb);
            __builtin_amdgcn_sched_barrier(0);
            compute_ktile<BITS, NTF, 1, 4>(ra, rb, sa, sb, kn, xa, ops, acc);
            ra.s2 = na.s2 | (na.s2 << 16);
            ra.m2 = na.m2 | (na.m2 << 16);
            rb.s2 = nb.s2 | (nb.s2 << 16);
            rb.m2 = nb.m2 | (nb.m2 << 16);
            __builtin_amdgcn_sched_barrier(0);
        } else {
            compute_ktile<BITS, NTF, 0, 4>(ra, rb, sa, sb, kn, xa, ops, acc);
        }
        if constexpr (kSecondSet) {
            adopt_strip<BITS>(ra, na);
            adopt_strip<BITS>(rb, nb);
            // finish the hand-over here, not after the next tile's requests
            // (a wait placed there would also wait for the copies just issued)
            __builtin_amdgcn_sched_barrier(0);
        }
        wait_lds_copies<ktile_loads<BITS>()>();
        __syncthreads();
        buf ^= 1;
        xa = xa0 + (uint32_t)(buf * kXsBufBytes);
    }

    // epilogue.  D layout: lane (ln, kb), register i -> weight row 8*(i/4) + 4*kb + i%4, token ln
    if constexpr (MODE == 2) {
        // Down projection: a lane holds, of its token's row, 4 consecutive outputs per register group: stored as they
        // are, one instruction would touch 32 rows with 32 bytes each.  The wavefront turns each fragment round in LDS
        // instead (the token tiles are done with: the loop's last barrier follows the last tile's arithmetic and the
        // last copy's wait): 32 rows of its 64 columns, 256 bytes + 16 of padding per row (the padding keeps both the
        // lane-per-row writes and the 16-lanes-per-row reads free of bank conflicts, and holds the row's pair index),
        // read back so that 16 lanes store one row's 256 contiguous bytes.  A wavefront's LDS accesses execute in
        // order, and the area is its own: no barrier.
        const uint32_t ebase = xs_base + (uint32_t)wave * kEpiWaveBytes;
        const long jbase = ((long)nblock * kGmWaves + wave) * 64;
        const int rsub = lane >> 4, chunk = lane & 15;
        const bool col_ok = strip_ok[chunk >> 3];
        const uint32_t wr = ebase + (uint32_t)ln * kEpiRowBytes + (uint32_t)kb * 16u;
#pragma unroll
        for (int tf = 0; tf < NTF; tf++) {
            const int trow = 32 * tf + ln;
            const int pair_w = (trow < rows) ? perm[row0 + trow] : -1;
#pragma unroll
            for (int s = 0; s < 2; s++)
#pragma unroll
                for (int g = 0; g < 4; g++) {
                    uint4 o;
                    o.x = __float_as_uint(acc[s][tf][4 * g + 0]);
                    o.y = __float_as_uint(acc[s][tf][4 * g + 1]);
                    o.z = __float_as_uint(acc[s][tf][4 * g + 2]);
                    o.w = __float_as_uint(acc[s][tf][4 * g + 3]);
                    lds_write16(wr + (uint32_t)(s * 128 + g * 32), o);
                }
            if (kb == 0) lds_write4(ebase + (uint32_t)ln * kEpiRowBytes + 256u, (uint32_t)pair_w);
#pragma unroll
            for (int j = 0; j < 8; j++) {
                const uint32_t ra = ebase + (uint32_t)(rsub + 4 * j) * kEpiRowBytes;
                const int pair = (int)lds_read4(ra + 256u);
                const uint4 v = lds_read16(ra + (uint32_t)chunk * 16u);
                if (pair >= 0 && col_ok)
                    *reinterpret_cast<uint4*>(oout + (long)pair * N + jbase + 4 * chunk) = v;
            }
        }
        return;
    }
#pragma unroll
    for (int tf = 0; tf < NTF; tf++) {
        const int trow = 32 * tf + ln;
        if (MODE == 1) {
            // SwiGLU; the 16-bit intermediate is written in the column order the
            // down projection of this expert reads (see perm8 / perm16)
            // The workgroup's four strips are 128 adjacent features: every wavefront writes its 64 bytes of each
            // row into LDS (272 bytes per row), and after one barrier the rows go out whole, 16 lanes per row.
            const uint32_t dst = xs_base + (uint32_t)trow * kEpiRowBytes + (uint32_t)wave * 64u;
            uint32_t pk[4][2];
#pragma unroll
            for (int g = 0; g < 4; g++) {
                float hv[4];
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const float a = acc[0][tf][4 * g + i];
                    const float u = acc[1][tf][4 * g + i];
                    hv[i] = a * __builtin_amdgcn_rcpf(1.0f + __expf(-a)) * u;
                }
                if constexpr (BITS == 16) {
                    pk[g][0] = f32_to_bf16_bits(hv[0]) | (f32_to_bf16_bits(hv[1]) << 16);
                    pk[g][1] = f32_to_bf16_bits(hv[2]) | (f32_to_bf16_bits(hv[3]) << 16);
                } else {
                    pk[g][0] = pack_half2(hv[0], hv[1]);
                    pk[g][1] = pack_half2(hv[2], hv[3]);
                }
            }
            if constexpr (BITS == 16 || BITS == 8) {
                // features f0 + 8g + 4kb .. +4, natural order
#pragma unroll
                for (int g = 0; g < 4; g++) lds_write8(dst + (uint32_t)(2 * (8 * g + 4 * kb)), make_uint2(pk[g][0], pk[g][1]));
            } else if constexpr (BITS == 4) {
                // group of 8 features e0..e7: this lane holds e(4kb..4kb+3); stored order is
                // e0,e4,e1,e5 | e2,e6,e3,e7: the two kb lanes trade one packed pair
#pragma unroll
                for (int g = 0; g < 4; g++) {
                    const uint32_t send = kb ? pk[g][0] : pk[g][1];          // kb0 gives (e2,e3), kb1 gives (e4,e5)
                    const uint32_t got = (uint32_t)__shfl_xor((int)send, 32, kWave);
                    const uint32_t lo = kb ? got : pk[g][0];                 // kb0: (e0,e1)  kb1: (e2,e3)
                    const uint32_t hi = kb ? pk[g][1] : got;                 // kb0: (e4,e5)  kb1: (e6,e7)
                    const uint32_t o0 = (lo & 0xffffu) | (hi << 16);
                    const uint32_t o1 = (lo >> 16) | (hi & 0xffff0000u);
                    lds_write8(dst + (uint32_t)(2 * (8 * g + 4 * kb)), make_uint2(o0, o1));
                }
            } else {
                // group of 16 features = register groups (g, g+1), g even: this lane holds
                // e(4kb+i) and e(8+4kb+i); stored order interleaves them at 8kb .. 8kb+7
                {
#pragma unroll
                    for (int g = 0; g < 4; g += 2) {
                        const uint32_t a01 = pk[g][0], a23 = pk[g][1], b01 = pk[g + 1][0], b23 = pk[g + 1][1];
                        uint4 o;
                        o.x = (a01 & 0xffffu) | (b01 << 16);
                        o.y = (a01 >> 16) | (b01 & 0xffff0000u);
                        o.z = (a23 & 0xffffu) | (b23 << 16);
                        o.w = (a23 >> 16) | (b23 & 0xffff0000u);
                        lds_write16(dst + (uint32_t)(2 * (8 * g + 8 * kb)), o);
                    }
                }
            }
        }
    }
    if (MODE == 1) {
        __syncthreads();
        const long f0 = (long)nblock * (32 * kGmWaves);
        const int chunk = tid & 15;                        // 8 features
        const bool col_ok = f0 + 8 * chunk < N;
        for (int r = tid >> 4; r < rows; r += kGmThreads / 16) {
            const uint4 v = lds_read16(xs_base + (uint32_t)r * kEpiRowBytes + (uint32_t)chunk * 16u);
            if (col_ok) *reinterpret_cast<uint4*>(hout + (long)(row0 + r) * N + f0 + 8 * chunk) = v;
        }
    }
}

template <int MODE>
__global__ __launch_bounds__(kGmThreads, 2) void gemm_kernel(
    const uint16_t* __restrict__ x_bf16, const uint16_t* __restrict__ x_h4,
    const uint16_t* __restrict__ x_h2, const uint16_t* __restrict__ x_h8,
    const uint16_t* __restrict__ hbuf_in,
    const uint8_t* __restrict__ bits, const dymoe_expert_fmt* __restrict__ table,
    const int32_t* __restrict__ plan, int P, int E, int k_route, int H, int F,
    uint16_t* __restrict__ hbuf_out, float* __restrict__ opair, int max_tiles)
{
    // two token-tile buffers; the swizzle works on the address bits inside a row
    extern __shared__ __attribute__((aligned(1024))) uint16_t xs_raw[];
    const uint32_t xs = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint16_t*)xs_raw;
    const PlanPtrs pp = plan_ptrs(const_cast<int32_t*>(plan), E, P);
    const int K = (MODE == 1) ? H : F;
    const int N = (MODE == 1) ? F : H;
    const int splits = (MODE == 2) ? pp.ntiles[kPlanSplits] : 1;
    // Which (column block, tile, K split) this workgroup takes.  Both launches are one-dimensional: workgroups go to the
    // 8 XCDs (each with an L2 of its own) in turn by launch index, L -> XCD c = L % 8, place j = L / 8 in that XCD's
    // sequence, and the units (a tile's rows over one K split) are handed out 8 at a time, all their column blocks,
    // before the next 8 (so the longest-first order of the tile list survives).  Inside such a group of 8 units x nblk
    // column blocks one of two things can be shared through an XCD's L2, and the plan says which pays:
    //  * the token rows (second GEMM): the column blocks of a unit all read the same rows of the intermediate.  XCD c
    //    takes unit c of the group in every column block.  Right when an expert has one tile, as in the Mixtral prefill
    //    (the second GEMM read 1.9 x its operands before);
    //  * the weights: tiles of ONE expert are neighbours in the list (equal cost keys keep the expert order) and read the
    //    same weight strips column block by column block.  The group's 8 x nblk (unit, column block) pairs are numbered
    //    column block first, q = 8 * column block + unit, and XCD c takes q in [c * nblk, (c + 1) * nblk): a column
    //    block's strips are then read by at most two XCDs instead of eight.  Right when experts have many tiles (routing
    //    with a few popular experts: the first GEMM of the 128-expert layer streamed 3.4 x its weights, at 5.9 TB/s).
    // The plan counts tiles and experts with tiles; weights are shared when there are at least twice as many tiles.
    int tile, bx, bz;
    {
        const int cols = (MODE == 1) ? 32 * kGmWaves : 64 * kGmWaves;
        const int nblk = (N + cols - 1) / cols;
        const int L = blockIdx.x, c = L & 7, j = L >> 3;
        const int g = j / nblk, sq = j - g * nblk;
        const bool share_weights = pp.ntiles[0] >= 2 * pp.ntiles[2];
        int unit;
        if (share_weights) {
            const int q = c * nblk + sq;
            bx = q >> 3;
            unit = 8 * g + (q & 7);
        } else if (MODE == 2) {
            bx = sq;
            unit = 8 * g + c;
        } else {
            // (first GEMM, one tile per expert: a tile per XCD would give each XCD one format, and the formats differ in
            // cost per tile; the tile's column blocks go round all XCDs instead, launch index = tile * nblk + column block)
            unit = L / nblk;
            bx = L - unit * nblk;
        }
        tile = unit / splits;
        bz = unit - tile * splits;
        if (tile >= max_tiles) return;
    }
    if (tile >= pp.ntiles[0]) return;
    const int e = pp.tiles[4 * tile + 0];
    const int row0 = pp.tiles[4 * tile + 1];
    const int rows = pp.tiles[4 * tile + 2];
    const int b = bits[e];
    const dymoe_expert_fmt ex = table[e];
    // split-K (second GEMM only): split bz takes K-tiles [bz*per, (bz+1)*per) and its own output slab
    const int nkt = K / kBK;
    const int per = (nkt + splits - 1) / splits;
    const int kt_begin = bz * per;
    const int kt_end = min(nkt, kt_begin + per);
    float* oz = opair + (size_t)bz * (size_t)P * (size_t)N;
    if (kt_begin >= kt_end) {
        // a split with no K-tiles still owns its slab: write zeros
        if (MODE == 2) {
            const int cols = 64 * kGmWaves;     // columns of this workgroup
            for (int i = threadIdx.x; i < rows * (cols / 4); i += kGmThreads) {
                const int r = i / (cols / 4), c = bx * cols + (i % (cols / 4)) * 4;
                if (c < N)
                    *reinterpret_cast<float4*>(oz + (size_t)pp.perm[row0 + r] * N + c) = make_float4(0.f, 0.f, 0.f, 0.f);
            }
        }
        return;
    }
    const uint16_t* act = (MODE != 1) ? hbuf_in : (b == 16 ? x_bf16 : (b == 8 ? x_h8 : (b == 4 ? x_h4 : x_h2)));
    const int ntf = (rows + 31) >> 5;
    // one instantiation per (precision, number of 32-token fragments): the
    // accumulators then sit in fixed registers for the whole K loop
#define DYMOE_TILE(BITS_, NTF_)                                                                      \
    gemm_tile<MODE, BITS_, NTF_>(act, pp.perm, k_route, ex, K, N, kt_begin, kt_end, row0, rows,      \
                                 bx, hbuf_out, oz, xs)
#define DYMOE_TILE_NTF(BITS_)                     \
    switch (ntf) {                                \
    case 1: DYMOE_TILE(BITS_, 1); break;          \
    case 2: DYMOE_TILE(BITS_, 2); break;          \
    case 3: DYMOE_TILE(BITS_, 3); break;          \
    case 4: DYMOE_TILE(BITS_, 4); break;          \
    default:                                      \
        if constexpr (BITS_ == 4 || BITS_ == 2) { \
            DYMOE_TILE(BITS_, 5);                 \
        } else {                                  \
            DYMOE_TILE(BITS_, 4);                 \
        }                                         \
        break;                                    \
    }
    if (b == 16) {
        DYMOE_TILE_NTF(16)
    } else if (b == 8) {
        DYMOE_TILE_NTF(8)
    } else if (b == 4) {
        DYMOE_TILE_NTF(4)
    } else {
        DYMOE_TILE_NTF(2)
    }
#undef DYMOE_TILE_NTF
#undef DYMOE_TILE
}

// ----------------------------------------------------------------------------
// Tiles of one fragment (up to 32 token rows): decode batches, where an expert meets a few tokens and the launch is a stream
// of weights.  In gemm_kernel the four wavefronts of a workgroup own different columns and share the token tile, one K-tile
// ahead: with int4 weights that is 33 KB in flight per compute unit (4.2 TB/s), and where the workgroups do not fill the chip,
// a microsecond per K-tile.  Here the wavefronts of a workgroup share their columns (two strips of 32 weight rows) and split
// the K-tiles: nothing is shared before the end, so there are no barriers and no LDS in the loop, a wavefront keeps the next
// K-tile's codes in registers and reads its token rows straight from the cache (a lane's 128 bytes of a row per K-tile), three
// workgroups share a compute unit, and a chain is a quarter as long.  At the end the four partial sums meet in LDS, in
// wavefront order.
constexpr int kSmThreads = 256;
constexpr int kSmWaves = kSmThreads / kWave;

template <int BITS>
struct SmallStrips {
    StripRaw<BITS> a, b;
};

// A strip's K-tiles as a base that is the same for the whole wavefront and this lane's 32-bit offset: the loads then take the
// base from scalar registers, where 64-bit addresses per lane and load would not fit beside the operands.
template <int BITS>
struct SmallSrc {
    const char* p;
    const char* s;            // scale, zero
    const char* z;
    uint32_t off;
    int kt_stride, c_stride;
};

template <int BITS>
__device__ __forceinline__ SmallSrc<BITS> small_src(const MatPtr& m, long nt, int K, int lane)
{
    SmallSrc<BITS> src;
    const long tile_row = nt * (K >> 7);
    src.s = reinterpret_cast<const char*>(m.s + tile_row * 64);
    src.z = reinterpret_cast<const char*>(m.z + tile_row * 64);
    src.off = (uint32_t)(lane * 16);
    src.c_stride = 1024;
    if constexpr (BITS == 16) {
        src.kt_stride = 8192;
        src.p = m.wt + tile_row * 8192;
        if (!m.wt) {
            src.p = reinterpret_cast<const char*>(m.w + nt * 32 * K);
            src.off = (uint32_t)((lane & 31) * K * 2 + 128 * (lane >> 5));
            src.kt_stride = 256;
            src.c_stride = 16;
        }
    } else {
        src.kt_stride = 512 * BITS;
        src.p = m.q + tile_row * (512 * BITS);
    }
    return src;
}

template <int BITS>
__device__ __forceinline__ uint4 small_chunk(const SmallSrc<BITS>& src, int kt, int c)
{
    if constexpr (BITS == 16) return load_global<uint4>(src.p + ((long)kt * src.kt_stride + c * src.c_stride) + src.off);
    else return load_global<uint4>(src.p + (long)kt * (512 * BITS) + src.off + c * 1024);
}

template <int BITS>
__device__ __forceinline__ void small_strip(const SmallSrc<BITS>& src, int kt, uint32_t off2, StripRaw<BITS>& raw)
{
    constexpr int kChunks = (BITS == 16) ? 8 : (BITS == 8 ? 4 : (BITS == 4 ? 2 : 1));
#pragma unroll
    for (int c = 0; c < kChunks; c++) raw.r[c] = small_chunk<BITS>(src, kt, c);
    if constexpr (BITS != 16) {
        raw.s2 = load_global<uint16_t>(src.s + (long)kt * 128 + off2);
        raw.m2 = load_global<uint16_t>(src.z + (long)kt * 128 + off2);
    }
}

template <int MODE, int BITS>
__device__ __forceinline__ void small_tile(const uint16_t* __restrict__ act, const int32_t* __restrict__ perm, int k_route,
                                           const dymoe_expert_fmt& ex, int K, int N, int kt_begin, int kt_end, int row0, int rows,
                                           int nblock, uint16_t* __restrict__ hout, float* __restrict__ oout, float* s_red)
{
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int ln = lane & 31, kb = lane >> 5;
    const long nt_a = (MODE == 1) ? nblock : 2L * nblock, nt_b = (MODE == 1) ? nblock : 2L * nblock + 1;
    const SmallSrc<BITS> sa = small_src<BITS>(mat_ptr(ex, MODE == 1 ? 0 : 2, BITS), nt_a, K, lane);
    const SmallSrc<BITS> sb = small_src<BITS>(mat_ptr(ex, MODE == 1 ? 1 : 2, BITS), nt_b, K, lane);
    const int n = kt_end - kt_begin;
    const int k0 = kt_begin + n * wave / kSmWaves, k1 = kt_begin + n * (wave + 1) / kSmWaves;
    float16_t acc[2];
#pragma unroll
    for (int s = 0; s < 2; s++)
#pragma unroll
        for (int i = 0; i < 16; i++) acc[s][i] = 0.0f;
    if (k0 < k1) {
        const int r = min(ln, rows - 1);                // rows past the last token re-read it: computed and dropped
        const long src_row = (MODE == 1) ? (long)(perm[row0 + r] / k_route) : (long)(row0 + r);
        const char* const xp = reinterpret_cast<const char*>(act);
        const uint32_t xoff = (uint32_t)(src_row * K * 2 + 128 * kb);       // < 4 GiB, checked by the launcher
        const uint32_t off2 = (uint32_t)(lane * 2);
        uint4 x[8];
#pragma unroll
        for (int c = 0; c < 8; c++) x[c] = load_global<uint4>(xp + (long)k0 * 256 + xoff + 16 * c);
        // the K-tile in `w` against x; x, and for bf16 and int8 w itself, are refilled from K-tile kn as soon as they have been used
        auto compute = [&](SmallStrips<BITS>& w, int kn) {
#pragma unroll
            for (int jj = 0; jj < 4; jj++) {
                uint4 a0, a1, b0, b1;
                strip_frags<BITS>(w.a, jj, a0, a1);
                strip_frags<BITS>(w.b, jj, b0, b1);
                acc[0] = mfma16<BITS>(a0, x[2 * jj], acc[0]);
                acc[1] = mfma16<BITS>(b0, x[2 * jj], acc[1]);
                acc[0] = mfma16<BITS>(a1, x[2 * jj + 1], acc[0]);
                acc[1] = mfma16<BITS>(b1, x[2 * jj + 1], acc[1]);
                x[2 * jj] = load_global<uint4>(xp + (long)kn * 256 + xoff + 32 * jj);
                x[2 * jj + 1] = load_global<uint4>(xp + (long)kn * 256 + xoff + 32 * jj + 16);
                if constexpr (BITS == 16) {
                    w.a.r[2 * jj] = small_chunk<16>(sa, kn, 2 * jj);
                    w.a.r[2 * jj + 1] = small_chunk<16>(sa, kn, 2 * jj + 1);
                    w.b.r[2 * jj] = small_chunk<16>(sb, kn, 2 * jj);
                    w.b.r[2 * jj + 1] = small_chunk<16>(sb, kn, 2 * jj + 1);
                } else if constexpr (BITS == 8) {
                    w.a.r[jj] = small_chunk<8>(sa, kn, jj);
                    w.b.r[jj] = small_chunk<8>(sb, kn, jj);
                }
                __builtin_amdgcn_sched_barrier(0x4);            // only SALU may cross
            }
        };
        // past the end the loads re-read the last K-tile instead of branching
        auto fetch = [&](SmallStrips<BITS>& w, int kt) {
            small_strip<BITS>(sa, min(kt, k1 - 1), off2, w.a);
            small_strip<BITS>(sb, min(kt, k1 - 1), off2, w.b);
            __builtin_amdgcn_sched_barrier(0);
        };
        SmallStrips<BITS> w0;
        fetch(w0, k0);
        if constexpr (BITS == 16) {
            for (int kt = k0; kt < k1; kt++) compute(w0, min(kt + 1, k1 - 1));
        } else if constexpr (BITS == 8) {
            for (int kt = k0; kt < k1; kt++) {
                const int kn = min(kt + 1, k1 - 1);
                adopt_strip<8>(w0.a, w0.a);
                adopt_strip<8>(w0.b, w0.b);
                uint32_t nx[4];
                nx[0] = load_global<uint16_t>(sa.s + (long)kn * 128 + off2);
                nx[1] = load_global<uint16_t>(sa.z + (long)kn * 128 + off2);
                nx[2] = load_global<uint16_t>(sb.s + (long)kn * 128 + off2);
                nx[3] = load_global<uint16_t>(sb.z + (long)kn * 128 + off2);
                compute(w0, kn);
                w0.a.s2 = nx[0]; w0.a.m2 = nx[1]; w0.b.s2 = nx[2]; w0.b.m2 = nx[3];
            }
        } else {
            SmallStrips<BITS> w1;
            auto step = [&](SmallStrips<BITS>& w, int kt) {
                adopt_strip<BITS>(w.a, w.a);
                adopt_strip<BITS>(w.b, w.b);
                compute(w, min(kt + 1, k1 - 1));
            };
            for (int kt = k0; kt < k1; kt += 2) {
                fetch(w1, kt + 1);
                step(w0, kt);
                if (kt + 1 >= k1) break;
                fetch(w0, kt + 2);
                step(w1, kt + 1);
            }
        }
    }
    // partial sums: [wavefront][register of strip a, then b][lane]
#pragma unroll
    for (int s = 0; s < 2; s++)
#pragma unroll
        for (int i = 0; i < 16; i++) s_red[((wave * 2 + s) * 16 + i) * kWave + lane] = acc[s][i];
    __syncthreads();
    // wavefront w finishes registers 4 w .. 4 w + 3 of both strips: weight rows 8 w + 4 kb + 0 .. 3, token ln
    float v[2][4];
#pragma unroll
    for (int s = 0; s < 2; s++)
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const float* const at = s_red + (s * 16 + 4 * wave + i) * kWave + lane;
            v[s][i] = ((at[0] + at[2048]) + at[4096]) + at[6144];
        }
    if constexpr (MODE == 2) {
        if (ln < rows) {
            float* const dst = oout + (long)perm[row0 + ln] * N + 64L * nblock + 8 * wave + 4 * kb;
            store_global(dst, make_float4(v[0][0], v[0][1], v[0][2], v[0][3]));
            store_global(dst + 32, make_float4(v[1][0], v[1][1], v[1][2], v[1][3]));
        }
        return;
    }
    // SwiGLU; the 16-bit intermediate in the column order that the down projection of this expert reads (perm8 / perm16), turned
    // round in LDS so that rows leave 64 bytes at a time
    uint16_t hb[4];
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const float h = v[0][i] * __builtin_amdgcn_rcpf(1.0f + __expf(-v[0][i])) * v[1][i];
        hb[i] = (uint16_t)(BITS == 16 ? f32_to_bf16_bits(h) : f16_bits((_Float16)h));
    }
    __syncthreads();                                    // the partial sums have been read
    uint16_t* const s_h = reinterpret_cast<uint16_t*>(s_red) + ln * 40;      // 32 features a row, padded to 80 bytes
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const int f = 8 * wave + 4 * kb + i;            // feature of the block's 32
        int at = f;
        if constexpr (BITS == 4) at = (f & ~7) + 2 * (f & 3) + ((f >> 2) & 1);
        else if constexpr (BITS == 2) at = (f & ~15) + 2 * (f & 7) + ((f >> 3) & 1);
        s_h[at] = hb[i];
    }
    __syncthreads();
    const int row = tid >> 2;
    if (tid < 128 && row < rows)
        *reinterpret_cast<uint4*>(hout + (long)(row0 + row) * N + 32L * nblock + 8 * (tid & 3)) =
            *reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(s_red) + row * 40 + 8 * (tid & 3));
}

template <int MODE>
__global__ __launch_bounds__(kSmThreads, 3) void gemm_small_kernel(
    const uint16_t* __restrict__ x_bf16, const uint16_t* __restrict__ x_h4, const uint16_t* __restrict__ x_h2,
    const uint16_t* __restrict__ x_h8, const uint16_t* __restrict__ hbuf_in, const uint8_t* __restrict__ bits,
    const dymoe_expert_fmt* __restrict__ table, const int32_t* __restrict__ plan, int P, int E, int k_route, int H, int F,
    uint16_t* __restrict__ hbuf_out, float* __restrict__ opair, int max_tiles)
{
    __shared__ __attribute__((aligned(16))) float s_red[kSmWaves * 2 * 16 * kWave];
    const PlanPtrs pp = plan_ptrs(const_cast<int32_t*>(plan), E, P);
    const int K = (MODE == 1) ? H : F, N = (MODE == 1) ? F : H;
    const int splits = (MODE == 2) ? pp.ntiles[kPlanSplits] : 1;
    const int nblk = N / ((MODE == 1) ? 32 : 64);
    const int unit = blockIdx.x / nblk, bx = blockIdx.x - unit * nblk;
    const int tile = unit / splits, bz = unit - tile * splits;
    if (tile >= max_tiles || tile >= pp.ntiles[0]) return;
    const int e = pp.tiles[4 * tile + 0], row0 = pp.tiles[4 * tile + 1], rows = pp.tiles[4 * tile + 2];
    const int b = bits[e];
    const dymoe_expert_fmt ex = table[e];
    const int nkt = K / kBK, per = (nkt + splits - 1) / splits;
    const int kt_begin = min(nkt, bz * per), kt_end = min(nkt, kt_begin + per);      // (a split without K-tiles writes zeros)
    float* const oz = opair + (size_t)bz * (size_t)P * (size_t)N;
    const uint16_t* act = (MODE != 1) ? hbuf_in : (b == 16 ? x_bf16 : (b == 8 ? x_h8 : (b == 4 ? x_h4 : x_h2)));
    if (b == 16) small_tile<MODE, 16>(act, pp.perm, k_route, ex, K, N, kt_begin, kt_end, row0, rows, bx, hbuf_out, oz, s_red);
    else if (b == 8) small_tile<MODE, 8>(act, pp.perm, k_route, ex, K, N, kt_begin, kt_end, row0, rows, bx, hbuf_out, oz, s_red);
    else if (b == 4) small_tile<MODE, 4>(act, pp.perm, k_route, ex, K, N, kt_begin, kt_end, row0, rows, bx, hbuf_out, oz, s_red);
    else small_tile<MODE, 2>(act, pp.perm, k_route, ex, K, N, kt_begin, kt_end, row0, rows, bx, hbuf_out, oz, s_red);
}

// y[t,j] = sum_slot w[t,slot] * (sum over K splits of o[z,pair,j])  (pairs of skipped experts omitted)
// Bound: the slabs' way from memory.  SLOTS slots' rows are requested together, whether or not their experts run (a row
// inside the slab that no workgroup wrote is read and not used): one after the other behind their experts' bit widths, a
// thread had 16 bytes in flight.  us, one slot at a time / together: 61 tokens x 8 slots of 2048 5.9 / 4.7, 24 x 2 of
// 4096 with three splits 5.5 / 4.8, 2048 x 8 of 2048 33.8 / 31.8 (a copy's rate).
template <int SLOTS>
__global__ __launch_bounds__(256) void gemm_combine_kernel(
    const float* __restrict__ opair, const int32_t* __restrict__ idx, const float* __restrict__ w,
    const uint8_t* __restrict__ bits, const int32_t* __restrict__ n_splits, int T, int H, int E, int k, int out_dtype,
    void* __restrict__ y)
{
    const int splits = *n_splits;
    const long i4 = (long)blockIdx.x * 256 + threadIdx.x;  // groups of 4 columns
    const long n4 = (long)T * (H >> 2);
    if (i4 >= n4) return;
    const int t = (int)(i4 / (H >> 2));
    const int j = (int)(i4 - (long)t * (H >> 2)) * 4;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int s0 = 0; s0 < k; s0 += SLOTS) {
        long p[SLOTS];
        int e[SLOTS];
        float g[SLOTS];
        float4 o[SLOTS];
#pragma unroll
        for (int u = 0; u < SLOTS; u++) {
            p[u] = (long)t * k + min(s0 + u, k - 1);
            e[u] = idx[p[u]];
            g[u] = w[p[u]];
            o[u] = load_global<float4>(opair + p[u] * H + j);
        }
        // the other slabs, two at a time where the registers leave wavefronts enough
        constexpr int kSlabs = SLOTS <= 4 ? 2 : 1;
        for (int z = 1; z < splits; z += kSlabs) {
            float4 oa[SLOTS], ob[SLOTS];
            const bool two = kSlabs == 2 && z + 1 < splits;
#pragma unroll
            for (int u = 0; u < SLOTS; u++) oa[u] = load_global<float4>(opair + ((long)z * T * k + p[u]) * H + j);
            if (two) {
#pragma unroll
                for (int u = 0; u < SLOTS; u++) ob[u] = load_global<float4>(opair + ((long)(z + 1) * T * k + p[u]) * H + j);
            }
#pragma unroll
            for (int u = 0; u < SLOTS; u++) {
                o[u].x += oa[u].x; o[u].y += oa[u].y; o[u].z += oa[u].z; o[u].w += oa[u].w;
                if (two) {
                    o[u].x += ob[u].x; o[u].y += ob[u].y; o[u].z += ob[u].z; o[u].w += ob[u].w;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < SLOTS; u++) {
            const int b = (e[u] >= 0 && e[u] < E) ? bits[e[u]] : 0;
            if (s0 + u < k && (b == 16 || b == 8 || b == 4 || b == 2)) {
                acc.x = fmaf(g[u], o[u].x, acc.x);
                acc.y = fmaf(g[u], o[u].y, acc.y);
                acc.z = fmaf(g[u], o[u].z, acc.z);
                acc.w = fmaf(g[u], o[u].w, acc.w);
            }
        }
    }
    if (out_dtype == DYMOE_OUT_F32) {
        *reinterpret_cast<float4*>(reinterpret_cast<float*>(y) + (long)t * H + j) = acc;
    } else {
        uint2 pk;
        pk.x = f32_to_bf16_bits(acc.x) | (f32_to_bf16_bits(acc.y) << 16);
        pk.y = f32_to_bf16_bits(acc.z) | (f32_to_bf16_bits(acc.w) << 16);
        *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(y) + (long)t * H + j) = pk;
    }
}

constexpr size_t kGemmLdsBytes = 2 * (size_t)kXsBufBytes;     // two token-tile buffers

// Once per device, at context creation, with that device current: the kernels use more dynamic LDS than the default limit.
int ffn_gemm_init()
{
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_kernel<1>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)kGemmLdsBytes) != hipSuccess ||
        hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_kernel<2>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)kGemmLdsBytes) != hipSuccess)
        return DYMOE_EHIP;
    return DYMOE_OK;
}

// Limits of the launch shapes below, checked by the entry point before anything is enqueued: tiles and workgroups, and the
// token rows, which are addressed through an unsigned 32-bit byte offset.
bool ffn_gemm_fits(int T, int H, int F, int E, int k)
{
    const size_t P = (size_t)T * (size_t)k;
    const size_t tiles = (size_t)ffn_most_tiles(T, E, k);
    if (tiles > 65535) return false;
    // every launch is one-dimensional, 8 * column blocks * ceil(units / 8) workgroups at most, and units are more than tiles only
    // while they are no more than four per compute unit (split_rule)
    const size_t nblk = ((size_t)(F > H ? F : H) + 32 * kGmWaves - 1) / (32 * kGmWaves);
    if (8 * nblk * (tiles + 1) >= ((size_t)1 << 31)) return false;
    if ((size_t)T * H * 2 >= ((size_t)1 << 32) || P * (size_t)F * 2 >= ((size_t)1 << 32)) return false;
    return true;
}

// The intermediate takes half of its area (16-bit values where the other path has fp32): the slabs start behind it.
static size_t slabs_offset(int T, int F, int k, const FfnLayout& L) { return L.hbuf + round256((size_t)T * k * F * 2); }

// Whether a GEMM of blocks x tiles workgroups takes gemm_small_kernel, tiles of one fragment given.  Two things cost it its lead:
// rounds, since every workgroup starts with a chain of dependent loads (plan -> expert -> pointers -> first rows, 3 us), and
// token rows, which every wavefront reads for itself where the other kernel shares them through LDS (32 rows of K are as many bytes
// as the int4 weights of a workgroup).  Up to a workgroup per compute unit it is ahead with any number of rows, up to two with
// two thirds of a fragment, beyond with a few.  Time of the small kernel over the large one's, 720 layers of 4 to 16 experts, by
// workgroups and pairs per expert:
//   first GEMM   4-8   8-12  12-17  17-25  25-32        second GEMM   4-8   8-12  12-17  17-25  25-32
//       256     0.66   0.67   0.68   0.73   0.80          up to 255  0.81   0.83   0.85   0.89   0.97
//       512     0.84   0.87   0.90   0.93   1.10           384-511   0.88   0.89   0.92   0.98   1.08
//       768     0.97   1.04   1.06   1.17   1.32               768   0.99   1.02   1.05   1.11   1.22
// (One pair or two per expert, second GEMM of 1280 workgroups: 0.96.)
static bool small_ahead(const dymoe_ctx* ctx, int T, int E, int k, long blocks, long most_rounds, long few)
{
    const long P = (long)T * k, tiles = E < P ? E : P, wgs = blocks * tiles, cu = ctx->num_cu;
    if (ffn_tile_rows(T, E, k) != kGemmTileSmall) return false;
    return wgs <= cu || (wgs <= 2 * cu && P <= 20 * tiles) || (wgs <= most_rounds * cu && P <= few * tiles);
}
static bool small_first(const dymoe_ctx* ctx, int T, int F, int E, int k) { return small_ahead(ctx, T, E, k, F / 32, 3, 6); }

// The second GEMM splits K as well.  Not where a few experts' long rows give the other kernel one and a half rounds of splits: there
// the bf16 expert's workgroups are what the launch waits for and a shorter chain does not help (us, large / small: 29 tokens x 2
// of 8, 2048 x 5248 13.4 / 15.1, 24 x 2 of 8, 4096 x 14336 61 / 66).
static bool small_second(const dymoe_ctx* ctx, int T, int H, int F, int E, int k)
{
    const long P = (long)T * k, tiles = E < P ? E : P;
    const long nblk = (H + 64 * kGmWaves - 1) / (64 * kGmWaves);
    if (tiles <= 16 && F >= 24 * kBK && 8 * nblk * tiles >= 3L * ctx->num_cu / 2) return false;
    return small_ahead(ctx, T, E, k, H / 64, 5, 8);
}

SplitRule split_rule(const dymoe_ctx* ctx, int T, int H, int F, int E, int k, const FfnLayout& L)
{
    const long P = (long)T * k;
    SplitRule r;
    r.small = small_second(ctx, T, H, F, E, k);
    r.nblk = r.small ? H / 64 : (H + 64 * kGmWaves - 1) / (64 * kGmWaves);
    r.n_kt = F / kBK;
    r.num_cu = ctx->num_cu;
    long most = (long)((L.xh - slabs_offset(T, F, k, L)) / ((size_t)P * H * 4));        // slabs the workspace holds
    const int least = r.small ? 2 * kSmWaves * kBK : 2 * kBK;                           // two K-tiles per chain at least
    if (most > F / least) most = F / least;
    // no more workgroups than 4 per compute unit if every expert has tokens (every one of them has a tile, and P / 128 more at most),
    // unless the small kernel's chains get too long (22 tokens x 4 of 30, 2048 x 4736: one split of 37 K-tiles 43.4 us, two 33.4)
    const long blocks = r.nblk * ((E < P ? E : P) + P / (2 * kGemmTileM));
    long room = 4L * r.num_cu / blocks;
    if (r.small && room < split_chains(r.n_kt)) room = split_chains(r.n_kt);
    if (most > room) most = room;
    r.max = (int)(most > 8 ? 8 : most < 1 ? 1 : most);
    return r;
}

int plan_launch(dymoe_ctx* ctx, const void* x, const int32_t* idx, const uint8_t* bits, const dymoe_expert_fmt* table, int T, int H,
                int E, int k, const SplitRule& splits, const FfnLayout& L, char* ws, hipStream_t st);

// planned: the workspace already holds the plan and the copies of x (rank_plan_launch)
int ffn_gemm_launch(dymoe_ctx* ctx, const void* x, const int32_t* idx, const float* w, const uint8_t* bits,
                    const dymoe_expert_fmt* table, int T, int H, int F, int E, int k,
                    int out_dtype, void* y, void* workspace, bool planned, hipStream_t st)
{
    const FfnLayout L = ffn_layout(T, H, F, E, k);
    const int P = T * k;
    if (!ffn_gemm_fits(T, H, F, E, k)) return DYMOE_ENOTSUP;
    char* ws = (char*)workspace;
    uint16_t* hbuf = reinterpret_cast<uint16_t*>(ws + L.hbuf);   // [P,F] 16-bit
    uint16_t* xh4 = reinterpret_cast<uint16_t*>(ws + L.xh);      // [T,H] fp16, int4 column order
    uint16_t* xh2 = xh4 + round256((size_t)T * H * 2) / 2;       // [T,H] fp16, int2 column order
    uint16_t* xh8 = xh2 + round256((size_t)T * H * 2) / 2;       // [T,H] fp16, natural column order (int8)
    float* opair = reinterpret_cast<float*>(ws + slabs_offset(T, F, k, L));
    int32_t* plan = reinterpret_cast<int32_t*>(ws + L.plan);
    const uint16_t* xb = (const uint16_t*)x;

    if (!planned) {
        const int rc = plan_launch(ctx, x, idx, bits, table, T, H, E, k, split_rule(ctx, T, H, F, E, k, L), L, ws, st);
        if (rc != DYMOE_OK) return rc;
    }
    // what the kernels after the plan take as the bit widths: the plan's copy, 0 where the table lacks the format
    const uint8_t* run_bits = reinterpret_cast<const uint8_t*>(plan_ptrs(plan, E, P).cursor);
    constexpr size_t kLdsBytes = kGemmLdsBytes;
    const int max_tiles = ffn_most_tiles(T, E, k);
    if (small_first(ctx, T, F, E, k)) {
        dymoe_launch(ctx, DYMOE_K_GEMM1, (gemm_small_kernel<1>), dim3((unsigned)((F / 32) * max_tiles)), dim3(kSmThreads), 0, st, xb, xh4,
                     xh2, xh8, (const uint16_t*)nullptr, run_bits, table, plan, P, E, k, H, F, hbuf, (float*)nullptr, max_tiles);
    } else {
        const int cols1 = 32 * kGmWaves;
        const int nblk1 = (F + cols1 - 1) / cols1;
        const dim3 g1((unsigned)(8 * nblk1 * ((max_tiles + 7) / 8)));
        dymoe_launch(ctx, DYMOE_K_GEMM1, (gemm_kernel<1>), g1, dim3(kGmThreads), kLdsBytes, st, xb, xh4, xh2, xh8,
                     (const uint16_t*)nullptr, run_bits, table, plan, P, E, k, H, F, hbuf, (float*)nullptr, max_tiles);
    }
    DYMOE_HIP_LAUNCH_CHECK();
    // The down projection has few output tiles: K is split so that the launch covers the chip.  Each split writes its own slab
    // of per-pair outputs and the combine kernel adds the slabs in a fixed order.  The plan chooses the number (it knows the
    // tiles); workgroups beyond it end at once.
    const SplitRule rule = split_rule(ctx, T, H, F, E, k, L);
    const int units = max_tiles * rule.max;
    if (rule.small) {
        dymoe_launch(ctx, DYMOE_K_GEMM2, (gemm_small_kernel<2>), dim3((unsigned)(rule.nblk * units)), dim3(kSmThreads), 0, st, xb, xh4,
                     xh2, xh8, hbuf, run_bits, table, plan, P, E, k, H, F, (uint16_t*)nullptr, opair, max_tiles);
    } else {
        const dim3 g2((unsigned)(8 * rule.nblk * ((units + 7) / 8)));
        dymoe_launch(ctx, DYMOE_K_GEMM2, (gemm_kernel<2>), g2, dim3(kGmThreads), kLdsBytes, st, xb, xh4, xh2, xh8, hbuf,
                     run_bits, table, plan, P, E, k, H, F, (uint16_t*)nullptr, opair, max_tiles);
    }
    DYMOE_HIP_LAUNCH_CHECK();
    const long n4 = (long)T * (H / 4);
    auto combine = [&](auto kernel) {
        dymoe_launch(ctx, DYMOE_K_GEMM_COMBINE, kernel, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, st, opair, idx, w, run_bits,
                     plan_ptrs(plan, E, P).ntiles + kPlanSplits, T, H, E, k, out_dtype, y);
    };
    if (k == 1) combine(gemm_combine_kernel<1>);
    else if (k == 2) combine(gemm_combine_kernel<2>);
    else if (k <= 4) combine(gemm_combine_kernel<4>);
    else combine(gemm_combine_kernel<8>);
    DYMOE_HIP_LAUNCH_CHECK();
    return DYMOE_OK;
}

}  // namespace dymoe
