// Token grouping of the grouped-GEMM path: counting sort of the (token, slot) pairs by expert and the list of tiles, by one
// workgroup, as device functions shared by the stand-alone plan kernel and the one that ranks the experts as well; and the
// fp16 copies of the activations that the launch's other workgroups make meanwhile.
#pragma once
#include "common.hpp"
#include "ffn_layout.hpp"

namespace dymoe {

// Tiles of one expert with c pairs at b bits: 128 rows each, the last one shorter.  For the int4 and int2 formats a
// last remainder of 1..32 rows is attached to the tile before it instead (5 fragments of 32 tokens, 160 rows): a
// remainder tile streams and dequantises the expert's whole weight matrices once more for a handful of tokens, which
// costs a third to a half of a full tile's time and all of its memory traffic.  (bf16 and int8 strips leave no
// registers for a fifth pair of accumulators.)
__device__ __forceinline__ bool plan_tall(int c, int b)
{
    const int r = c % kGemmTileM;
    return (b == 4 || b == 2) && c > kGemmTileM && r >= 1 && r <= kGemmTileTall - kGemmTileM;
}
__device__ __forceinline__ int plan_tiles_of(int c, int b, int tile_m)
{
    const int lg = tile_m == kGemmTileM ? 7 : 5;
    static_assert(kGemmTileM == 1 << 7 && kGemmTileSmall == 1 << 5, "tiles of 128 or 32 rows");
    return ((c + tile_m - 1) >> lg) - (tile_m == kGemmTileM && plan_tall(c, b) ? 1 : 0);
}

// ints: counts[E] | offsets[E+1] | cursor[E] | ntiles (8 ints) | perm[P] | tiles[4*max_tiles] | draft[4*max_tiles]
// (cursor: its first E BYTES hold the bit width every expert is run at, which is bits[e] unless the table lacks that
// format, then 0; the GEMM and combine kernels read these instead of bits[])
struct PlanPtrs {
    int32_t* counts;
    int32_t* offsets;
    int32_t* cursor;
    int32_t* ntiles;
    int32_t* perm;
    int32_t* tiles;
};

__host__ __device__ inline PlanPtrs plan_ptrs(int32_t* base, int E, int P)
{
    PlanPtrs p;
    p.counts = base;
    p.offsets = p.counts + E;
    p.cursor = p.offsets + E + 1;
    p.ntiles = p.cursor + E;
    p.perm = p.ntiles + 8;
    p.tiles = p.perm + P;
    return p;
}

// Column order in which the code fields of a dword come out of the mask-and-or
// extraction: inside every 8 columns (int4) 0,4,1,5,2,6,3,7; inside every 16
// columns (int2) 0,8,1,9,...,7,15.  Inputs are packed pairs of 16-bit values.
__device__ __forceinline__ uint4 perm8(const uint4 v)
{
    uint4 o;
    o.x = (v.x & 0xffffu) | (v.z << 16);
    o.y = (v.x >> 16) | (v.z & 0xffff0000u);
    o.z = (v.y & 0xffffu) | (v.w << 16);
    o.w = (v.y >> 16) | (v.w & 0xffff0000u);
    return o;
}

__device__ __forceinline__ void perm16(const uint4 a, const uint4 b, uint4& o0, uint4& o1)
{
    o0.x = (a.x & 0xffffu) | (b.x << 16);
    o0.y = (a.x >> 16) | (b.x & 0xffff0000u);
    o0.z = (a.y & 0xffffu) | (b.y << 16);
    o0.w = (a.y >> 16) | (b.y & 0xffff0000u);
    o1.x = (a.z & 0xffffu) | (b.z << 16);
    o1.y = (a.z >> 16) | (b.z & 0xffff0000u);
    o1.z = (a.w & 0xffffu) | (b.w << 16);
    o1.w = (a.w >> 16) | (b.w & 0xffff0000u);
}

// Three fp16 copies of the bf16 activations (exact inside fp16's normal range):
// one in each of the column orders above and one in the natural order (int8
// codes come out of a dword in order).  A thread converts 16 columns.  A copy nobody will read is left out (NULL).
__device__ __forceinline__ void prep_x(const uint16_t* __restrict__ x, long i, uint16_t* __restrict__ xh4,
                                       uint16_t* __restrict__ xh2, uint16_t* __restrict__ xh8)
{
    const uint4 a = reinterpret_cast<const uint4*>(x)[2 * i];
    const uint4 b = reinterpret_cast<const uint4*>(x)[2 * i + 1];
    uint4 ha, hb;
    ha.x = pack_half2(bf16_lo(a.x), bf16_hi(a.x)); ha.y = pack_half2(bf16_lo(a.y), bf16_hi(a.y));
    ha.z = pack_half2(bf16_lo(a.z), bf16_hi(a.z)); ha.w = pack_half2(bf16_lo(a.w), bf16_hi(a.w));
    hb.x = pack_half2(bf16_lo(b.x), bf16_hi(b.x)); hb.y = pack_half2(bf16_lo(b.y), bf16_hi(b.y));
    hb.z = pack_half2(bf16_lo(b.z), bf16_hi(b.z)); hb.w = pack_half2(bf16_lo(b.w), bf16_hi(b.w));
    if (xh4) {
        reinterpret_cast<uint4*>(xh4)[2 * i] = perm8(ha);
        reinterpret_cast<uint4*>(xh4)[2 * i + 1] = perm8(hb);
    }
    if (xh2) {
        uint4 o0, o1;
        perm16(ha, hb, o0, o1);
        reinterpret_cast<uint4*>(xh2)[2 * i] = o0;
        reinterpret_cast<uint4*>(xh2)[2 * i + 1] = o1;
    }
    if (xh8) {
        reinterpret_cast<uint4*>(xh8)[2 * i] = ha;
        reinterpret_cast<uint4*>(xh8)[2 * i + 1] = hb;
    }
}


constexpr int kPlanThreads = 1024;     // one workgroup of 16 wavefronts
constexpr int kPlanWaves = kPlanThreads / kWave;
constexpr int kPlanPrivE = 256;        // a histogram per wavefront: 16 x 256 counters = 16 KiB
constexpr int kPlanShortList = 1024;   // tiles of a list that a thread each ranks

// Per expert: its pairs (returned), and in its wavefronts' counters the position of each one's first among them.
__device__ __forceinline__ int plan_gather(int e, int E, int32_t* s_priv)
{
    int c[kPlanWaves], run = 0;
#pragma unroll
    for (int wv = 0; wv < kPlanWaves; wv++) c[wv] = s_priv[wv * E + e];
#pragma unroll
    for (int wv = 0; wv < kPlanWaves; wv++) {
        s_priv[wv * E + e] = run;
        run += c[wv];
    }
    return run;
}

// Number of K splits of the second GEMM: nblk column blocks, n_kt K-tiles, up to max splits, num_cu compute units that hold two
// workgroups each (small: of the kernel for tiles of one fragment, which holds three).
struct SplitRule {
    int nblk, n_kt, max, num_cu;
    bool small;
};
constexpr int kPlanSplits = 3;         // where the plan keeps it, behind the tile counts

__host__ __device__ inline int split_chains(int n_kt) { return (n_kt + 12) / 24; }

// In units of a round of two unsplit workgroups per compute unit, n workgroups per compute unit of 1 / s of the K-tiles each take
// 0.7 / s up to one (each has a unit to itself), (0.67 + 0.2 n) / s up to two (one round) and (0.25 + 0.5 n) / s beyond; every
// split writes and reads a slab, 0.011 (0.4 + rows per tile / 128) per workgroup and K-tile.  Over 437 layers of 5 to 2100
// tokens with a choice, every number timed, GEMM and combine are 1.0 % off the best on average, 12 of them more than 10 %
// (always 3 num_cu / blocks splits for tiles of one fragment, else 0.6 / 1 / 0.3 + 0.5 n and 0.0147 whatever the rows: 1.8 %, 31 of
// them).  us: 512 tokens of the Mixtral shape (8 tiles x 16 blocks) 2 splits 181, 4 138 (9 x 16: 1 328, 2 209, 3 170, 4 189); 172 x 6
// of 3328 x 3072 (17 x 13) 1 74, 2 54; 1743 x 2 of 768 x 5120 (31 x 3) 1 101, 2 62, 3 56, 4 51, 5 50, 6 53; 187 x 2 of 512 x 7168
// (63 x 2, one fragment) 4 32, 6 38.
// With a 16-bit expert among tiles of one fragment, which stream weights of very different widths, one and a half rounds of
// workgroups level them out (24 tokens of the Mixtral shape, 8 x 16: 2 splits 87, 4 86, 5 73, 6 67, 8 69).
// The kernel for tiles of one fragment splits K over its wavefronts already: about 24 K-tiles per split at most (split_chains), so
// that a bf16 expert's workgroups do not outlast the launch (80 tokens of 512 x 4864: 25.4 us with 38, 21.3 with 19).
// By one wavefront, a lane per number (max <= 64); the least cost, the smaller number of equals.  wide: tiles of 16-bit experts.
__device__ __forceinline__ void plan_splits(int tiles, int pairs, bool wide, const SplitRule& r, const PlanPtrs& pp)
{
    const int lane = threadIdx.x & (kWave - 1), s = lane + 1;
    const int blocks = max(1, r.nblk * tiles);
    int best = 1;
    if (r.max > 1) {
        if (r.small || (wide && pairs <= 32 * tiles)) {
            best = 3 * r.num_cu / blocks;
            if (r.small) best = max(best, split_chains(r.n_kt));
            best = max(1, min(r.max, best));
        } else {
            const float per_cu = (float)(blocks * s) / (float)r.num_cu;
            const float rounds = per_cu <= 1.0f ? 0.7f : per_cu <= 2.0f ? 0.67f + 0.2f * per_cu : 0.25f + 0.5f * per_cu;
            const float slab = 0.011f * (0.4f + (float)pairs / (128.0f * (float)max(1, tiles)));
            const float cost = s <= r.max ? rounds / (float)s + slab * (float)blocks * (float)s / (float)r.n_kt : 1e30f;
            best = __ffsll((long long)__ballot(cost == -wave_max_dpp(-cost)));
        }
    }
    if (lane == 0) pp.ntiles[kPlanSplits] = best;
}

// s_count, s_bits: pairs and bit width of every expert (no pairs where it does not run) -> first pair and first tile of
// each, the totals to memory.  The caller's s_count and s_bits are visible to all; so are the results.
__device__ __forceinline__ void plan_scan(int E, int tile_m, const int32_t* s_count, const uint8_t* s_bits, int32_t* s_off, int32_t* s_tile0,
                                          const SplitRule& splits, const PlanPtrs& pp)
{
    const int tid = threadIdx.x, wave = tid / kWave;
    // E is at most 1024: one wavefront walks the experts in strides
    if (wave == 0) {
        const int lane = tid;
        int run = 0, trun = 0, with_tiles = 0;
        for (int e0 = 0; e0 < E; e0 += kWave) {
            const int e = e0 + lane;
            const int c = (e < E) ? s_count[e] : 0;
            const int nt_e = (e < E) ? plan_tiles_of(c, s_bits[e], tile_m) : 0;
            const int incl = wave_scan_dpp_i32(c), tincl = wave_scan_dpp_i32(nt_e);
            if (e < E) {
                s_off[e] = run + incl - c;
                s_tile0[e] = trun + tincl - nt_e;
            }
            run += __builtin_amdgcn_readlane(incl, kWave - 1);
            trun += __builtin_amdgcn_readlane(tincl, kWave - 1);
            with_tiles += __popcll(__ballot(nt_e > 0));
        }
        if (lane == 0) {
            s_off[E] = run;
            s_tile0[E] = trun;
            pp.ntiles[0] = trun;
            pp.ntiles[1] = run;
            pp.ntiles[2] = with_tiles;      // experts with at least one tile (the GEMM launches pick their XCD mapping by it)
        }
    }
    bool wide = false;                          // (meanwhile)
    if (wave == kPlanWaves - 1)
        for (int e = tid & (kWave - 1); e < E; e += kWave) wide |= s_count[e] > 0 && s_bits[e] == 16;
    __syncthreads();
    if (wave == kPlanWaves - 1) plan_splits(s_tile0[E], s_off[E], __any(wide), splits, pp);
}

// Cost key of a tile, roughly the time a workgroup spends on it: streaming (bf16) or dequantising (int4, int2) the weights
// costs the same whatever the number of tokens; the MFMA work grows with the 32-token fragments.
__device__ __forceinline__ int plan_tile_key(int b, int rows) { return (b == 16 ? 100 : (b == 2 ? 60 : 61)) + 10 * ((rows + 31) >> 5); }
// The keys' order in four bits: 70, 71 (one fragment: int2; int4 and int8) -> 0, 1; 80, 81 -> 2, 3; .. 140 (bf16, four) -> 14.
__device__ __forceinline__ int plan_key_order(int key) { return 2 * ((key - 70) / 10) + (key % 10); }
constexpr int kPlanOrders = 16;

// The tile list, longest first: workgroups are dispatched in tile order, so the cheap tiles (few tokens) fill the end of
// the launch instead of stretching it.  Order: key descending, then position ascending (the tiles of an expert stay together).
// A thread per tile finds its expert and counts, among its wavefront's, the tiles of its key before it; the wavefronts'
// counts, by key and then by wavefront, are scanned by one wavefront.  s_cnt: 256 counters, 16-byte aligned.  Up to 1024 tiles.
// (197 tiles of the 128-expert layer: 1.3 us; ranked by comparing every tile with every other, a wavefront per tile, 5.4 us.)
__device__ __forceinline__ void plan_tile_list(int E, int tile_m, const int32_t* s_count, const uint8_t* s_bits, const int32_t* s_off,
                                               const int32_t* s_tile0, int32_t* s_cnt, const PlanPtrs& pp)
{
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int nt_all = s_tile0[E];
    if (tid < kPlanOrders * kPlanWaves) s_cnt[tid] = 0;
    __syncthreads();
    int4 rec = make_int4(0, 0, 0, 0);
    int at = -1, turn = 0;                      // at: the tile's counter
    if (wave * kWave < nt_all) {
        if (tid < nt_all) {
            int e = 0;                          // the last expert whose first tile is not behind this one
            for (int step = E > 64 ? 512 : 32; step > 0; step >>= 1)
                if (e + step < E && s_tile0[e + step] <= tid) e += step;
            const int m0 = (tid - s_tile0[e]) * tile_m;
            rec.x = e;
            rec.y = s_off[e] + m0;
            rec.z = (tid + 1 == s_tile0[e + 1]) ? s_count[e] - m0 : tile_m;     // (the last tile: up to 160 rows when tall)
            rec.w = plan_tile_key(s_bits[e], rec.z);
            at = (kPlanOrders - 1 - plan_key_order(rec.w)) * kPlanWaves + wave;
        }
        unsigned long long left = __ballot(at >= 0);
        while (left) {                          // key by key
            const int one = __builtin_amdgcn_readlane(at, __ffsll((long long)left) - 1);
            const unsigned long long same = __ballot(at == one);
            if (at == one) {
                turn = __popcll(same & ((1ull << lane) - 1));
                if (turn == 0) s_cnt[at] = __popcll(same);
            }
            left &= ~same;
        }
    }
    __syncthreads();
    if (wave == 0) {
        int4* const c4 = reinterpret_cast<int4*>(s_cnt) + lane;
        const int4 c = *c4;
        const int before = wave_scan_dpp_i32(c.x + c.y + c.z + c.w) - (c.x + c.y + c.z + c.w);
        *c4 = make_int4(before, before + c.x, before + c.x + c.y, before + c.x + c.y + c.z);
    }
    __syncthreads();
    if (at >= 0) {
        int32_t* const dst = pp.tiles + 4 * (s_cnt[at] + turn);
        dst[0] = rec.x; dst[1] = rec.y; dst[2] = rec.z; dst[3] = rec.w;
    }
}

// The same for lists of more than 1024 tiles: laid out in memory (draft) by a thread per expert, every tile's position by
// comparison with all others, a wavefront per tile.
__device__ __forceinline__ void plan_tile_list_long(int E, int tile_m, const int32_t* s_count, const uint8_t* s_bits, const int32_t* s_off,
                                                    const int32_t* s_tile0, int32_t* draft, const PlanPtrs& pp)
{
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid & (kWave - 1);
    const int nt_all = s_tile0[E];
    for (int e = tid; e < E; e += kPlanThreads) {
        const int c = s_count[e], b = s_bits[e];
        int nt = s_tile0[e];
        const int nt_end = s_tile0[e + 1];
        for (int m0 = 0; nt < nt_end; m0 += tile_m, nt++) {
            const int rows = (nt == nt_end - 1) ? c - m0 : tile_m;
            draft[4 * nt + 0] = e;
            draft[4 * nt + 1] = s_off[e] + m0;
            draft[4 * nt + 2] = rows;
            draft[4 * nt + 3] = plan_tile_key(b, rows);
        }
    }
    __syncthreads();        // (workgroup-wide visibility of the draft)
    for (int i = wave; i < nt_all; i += kPlanWaves) {
        const int key = draft[4 * i + 3];
        int pos = 0;        // the same in every lane: each stride of 64 tiles adds the number of its lanes that precede i
        for (int j0 = 0; j0 < nt_all; j0 += kWave) {
            const int j = j0 + lane;
            const int kj = (j < nt_all) ? draft[4 * j + 3] : -1;
            pos += __popcll(__ballot(j < nt_all && (kj > key || (kj == key && j < i))));
        }
        if (lane < 4) pp.tiles[4 * pos + lane] = draft[4 * i + lane];
    }
}

__device__ __forceinline__ void plan_tables(int E, const int32_t* s_count, const uint8_t* s_bits, const int32_t* s_off, const PlanPtrs& pp)
{
    for (int e = threadIdx.x; e < E; e += kPlanThreads) {
        pp.counts[e] = s_count[e];
        pp.offsets[e] = s_off[e];
        reinterpret_cast<uint8_t*>(pp.cursor)[e] = (s_bits[e] & 0x80) ? 0 : s_bits[e];
    }
    if (threadIdx.x == 0) pp.offsets[E] = s_off[E];
}

}  // namespace dymoe
