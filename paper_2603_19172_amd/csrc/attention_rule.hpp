// Which kernels the attention-derived token score takes for a size (attention.hip): host code only.
#pragma once
#include <cmath>
#include <limits>

namespace dymoe {

constexpr int kAtWaves = 4;         // wavefronts of a workgroup of the narrow pair

// Which pair of kernels, by what each is expected to take.  Narrow: a workgroup per 32-token fragment, its wavefronts sharing the streamed
// tokens (many workgroups, operands straight from global memory).  Wide: blocks of 128 or 256 tokens with the stream in LDS.  The
// numbers are those of the whole score in us, fitted to 372 sizes a head size (1 to 64 heads of 257 to 8000 tokens, both masks;
// errors 3 to 5 % rms, the narrow pair's in the range where it matters), so that the pair taken is 0.1 % (d = 128) and 0.2 % slower
// than the best of them on average, 4 and 7 % at worst; with lines drawn at fragment counts alone it was 1.4 % and more, up to half.
struct AtChoice {
    int owners;                 // 0: the narrow pair, else tokens per block of the wide pair, in units of 64
    int waves;                  // wavefronts of a workgroup
};
struct AtCost {
    AtChoice form;
    int resident;               // blocks at a time on a compute unit
    double start;               // launches, score kernel, ends of both passes
    double block;               // a block's own start and end
    double alone, shared;       // a streamed fragment of a block's chain; of each of several blocks beside each other
    double even, pairs;         // causal: what an uneven end adds, and with no more than two blocks a place (the longest with the shortest)
};

// Unmasked, all blocks are alike and go over the chip in rounds; causal blocks come longest first and fill it evenly, unless the
// longest alone takes longer.
inline double attn_wide_us(int nfrag, int n_heads, int causal, int num_cu, const AtCost& c)
{
    const int owners = c.form.owners, streams = c.form.waves / owners;
    const double blocks = (double)((nfrag + 2 * owners - 1) / (2 * owners)) * n_heads;
    const double chain = (nfrag + streams - 1) / streams, places = (double)num_cu * c.resident;
    if (causal)
        return c.start + std::fmax(c.block + chain * c.alone, (blocks > 2.0 * places ? c.even : c.pairs) +
                                                                  blocks / num_cu * (c.block / c.resident + 0.5 * chain * c.shared));
    auto round = [&](double beside) { return beside > 0.0 ? c.block + chain * std::fmax(c.alone, beside * c.shared) : 0.0; };
    const double whole = std::floor(blocks / places);
    return c.start + whole * round(c.resident) + round(std::ceil((blocks - whole * places) / num_cu));
}

// The narrow pair's workgroups are all resident where it is in question (up to five a compute unit): a unit takes the longest one's
// chain, a memory latency per fragment (`alone`), or the products of all that it holds (`shared` per fragment and half of that per workgroup).  Under the causal mask
// that depends on which fragments meet on a unit: where the fragments of a head divide its turn, one holds nothing but last ones
// (512 tokens x 64 heads 26.4 us, wide 18.7; 700 x 24 18.3 and 21.2 with as many per unit).
inline double attn_narrow_us(int nfrag, int n_heads, int causal, int num_cu, double start, double alone, double shared)
{
    const long all = (long)nfrag * n_heads;
    if (all > 5L * num_cu) return std::numeric_limits<double>::infinity();
    const int chain = (nfrag + kAtWaves - 1) / kAtWaves;
    if (all <= num_cu) return start + chain * alone;
    if (!causal) return start + std::fmax(chain * alone, (double)((all + num_cu - 1) / num_cu) * (chain + 0.5) * shared);
    // the narrow kernels' order, one XCD of it where the heads divide: a workgroup a unit in turn
    const bool whole_heads = n_heads % 8 == 0 && num_cu >= 8;
    int load[512] = {}, most = 0;
    const int heads = whole_heads ? n_heads / 8 : n_heads;
    const int units = (whole_heads ? num_cu / 8 : num_cu) < 512 ? (whole_heads ? num_cu / 8 : num_cu) : 512;
    for (int h = 0, at = 0; h < heads; h++)
        for (int f = 0; f < nfrag; f++) {
            load[at] += 2 * (f / kAtWaves) + 3;                         // in half fragments
            most = load[at] > most ? load[at] : most;
            if (++at == units) at = 0;
        }
    return start + std::fmax(chain * alone, 0.5 * most * shared);
}

// Whole score, us, narrow / blocks of 128 / of 256 tokens (d = 128) or three at a time of 128 on a unit (d = 64):
//                    d = 128, causal           unmasked              d = 64, causal            unmasked
//     512 x 20   26.1 / 19.3 / 28.2     27.2 / 18.2 / 24.5     16.6 / 17.6 / 17.8     16.7 / 16.1 / 15.9
//    1000 x  8   26.9 / 27.6 / 42.9     27.4 / 26.4 / 39.6     16.3 / 24.0 / 26.0     17.0 / 22.7 / 24.2
//    1200 x  8   33.5 / 31.4 / 48.3     44.8 / 30.6 / 45.3     19.9 / 26.7 / 29.7     26.7 / 25.6 / 28.0
//    2048 x  8   57.0 / 43.0 / 70.0     68.7 / 41.9 / 66.9     31.6 / 35.7 / 40.6     38.6 / 34.4 / 38.9
//    4096 x  1   81.9 / 73.5 / 126      83.5 / 72.4 / 122      39.9 / 58.6 / 69.8     41.1 / 57.6 / 67.5
//    1400 x 48   134 / 58.1 / 55.1      203 / 96.1 / 99.9      68.8 / 48.7 / 36.8     106 / 74.2 / 55.7
//    4096 x 48   809 / 274 / 251        1414 / 475 / 423       426 / 207 / 153        723 / 340 / 278
// (256 tokens a block at d = 64 are nowhere the fastest.)
inline AtChoice attn_choice(int nfrag, int n_heads, int causal, int head_dim, int num_cu)
{
    const AtChoice none = {0, kAtWaves};
    if (nfrag < 9) return none;         // 64 tokens x 192 heads 14.7 / 19.6, 200 x 64 16.4 / 18.4, 300 x 64 27.6 / 21.7 (d = 128)
    static constexpr AtCost d128[] = {{{2, 8}, 1, 1.6, 9.2, 2.06, 2.06, 14.0, 5.5}, {{4, 8}, 1, 0.0, 12.25, 1.885, 1.885, 13.3, 9.7}};
    static constexpr AtCost d64[] = {{{2, 8}, 1, 4.5, 6.5, 1.52, 1.52, 13.7, 7.2}, {{2, 4}, 3, 6.1, 3.95, 0.97, 0.73, 9.4, 9.4}};
    double best = head_dim == 128 ? attn_narrow_us(nfrag, n_heads, causal, num_cu, 7.6, 2.34, 1.84)
                                  : attn_narrow_us(nfrag, n_heads, causal, num_cu, 8.0, 1.03, 0.92);
    AtChoice choice = none;
    for (const AtCost& c : head_dim == 128 ? d128 : d64) {
        const double us = attn_wide_us(nfrag, n_heads, causal, num_cu, c);
        if (us < best) {
            best = us;
            choice = c.form;
        }
    }
    return choice;
}

}  // namespace dymoe
