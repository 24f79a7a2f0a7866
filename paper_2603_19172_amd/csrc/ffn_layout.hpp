// Workspace layout of dymoe_moe_ffn_mixed (host side, shared by the size query
// and the two FFN paths).
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace dymoe {

constexpr int kSeg = 2048;        // columns one wavefront covers per GEMV row segment
constexpr int kGemmTileM = 128;   // token rows per grouped-GEMM tile
constexpr int kGemmTileTall = 160; // the last tile of an int4 / int2 expert also takes a remainder of up to 32 rows
constexpr int kPlanTileMin = 32;  // sizing granularity of the tile list

// Token rows per grouped-GEMM tile.  Few tokens per expert: tiles of one 32-row fragment, for the kernel that streams weights
// with all four wavefronts of a workgroup on the same columns.
constexpr int kGemmTileSmall = 32;
static inline int ffn_tile_rows(int T, int E, int k)
{
    return (T <= 32 || (T <= 128 && (long)T * k <= 8L * E)) ? kGemmTileSmall : kGemmTileM;
}

// Tiles of T * k pairs at most: one of every expert with pairs is not whole.
static inline int ffn_most_tiles(int T, int E, int k)
{
    const long P = (long)T * k;
    return (int)(P / ffn_tile_rows(T, E, k) + (E < P ? E : P));
}

struct FfnLayout {
    size_t hbuf;    // [P,F] SwiGLU intermediate: fp32 (GEMV) or 16-bit (GEMM; the splits' output slabs start right behind it)
    size_t part;    // room for [P,H] fp32 per-pair outputs, one slab per split (GEMV: the pairs' entries, or the fused front end's logits)
    size_t xh;      // GEMM: three [T,H] fp16 copies of the activations (int4 / int2 / natural column order); fused GEMV: the pairs' entries
    size_t plan;    // int32: counts[E], offsets[E+1], cursor[E], ntiles, perm[P], tiles[4*maxtiles], draft[4*maxtiles]
    size_t total;
    int max_tiles;
};

static inline size_t round256(size_t v) { return (v + 255) & ~(size_t)255; }

static inline FfnLayout ffn_layout(int T, int H, int F, int E, int k)
{
    FfnLayout L;
    size_t P = (size_t)T * (size_t)k;
    size_t nseg = ((size_t)F + kSeg - 1) / kSeg;
    L.max_tiles = (int)(P / kPlanTileMin + (size_t)E + 1);
    L.hbuf = 0;
    L.part = L.hbuf + round256(P * (size_t)F * 4);
    L.xh = L.part + round256(P * nseg * (size_t)H * 4);
    L.plan = L.xh + 3 * round256((size_t)T * (size_t)H * 2);
    size_t plan_ints = (size_t)E + ((size_t)E + 1) + (size_t)E + 8 + P + 8 * (size_t)L.max_tiles;
    L.total = L.plan + round256(plan_ints * 4);
    return L;
}

}  // namespace dymoe
