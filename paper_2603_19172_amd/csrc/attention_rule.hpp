// Which kernels the attention-derived token score takes for a size (attention.hip): host code only.
#pragma once
#include <cmath>
#include <limits>

namespace dymoe {

constexpr int kAtWaves = 4;         // wavefronts of a workgroup of the narrow pair

// Blocks of the wide pair that a compute unit holds at a time: eight wavefronts fill it, of four as many as registers and LDS take.
constexpr int at_resident(int head_dim, int waves) { return waves == 8 ? 1 : head_dim == 64 ? 3 : 2; }

// Which pair of kernels, by what each is expected to take.  Narrow: a workgroup per 32-token fragment, its wavefronts sharing the streamed
// tokens (many workgroups, operands straight from global memory).  Wide: blocks of 128 or 256 tokens with the stream in LDS.  The
// numbers are those of the whole score in us, fitted to 804 sizes a head size (1 to 96 heads of 257 to 8000 tokens, both masks;
// errors 4 to 8 % rms), so that the pair taken is 0.2 % (d = 128) and 0.1 % slower than the best of them on average, 9 and 6 % at
// worst; with lines drawn at fragment counts alone it was 1.4 % and more, up to half.
struct AtChoice {
    int owners;                 // 0: the narrow pair, else tokens per block of the wide pair, in units of 64
    int waves;                  // wavefronts of a workgroup
};
struct AtCost {
    AtChoice form;
    double start;               // launches, score kernel, ends of both passes
    double block;               // a block's own start and end
    double alone, shared;       // a streamed fragment of a block's chain; of each of several blocks beside each other
    double even, pairs;         // causal: what an uneven end adds, and with no more than two blocks a place (the longest with the shortest)
};

// Unmasked, all blocks are alike and go over the chip in rounds; causal blocks come longest first and fill it evenly, unless the
// longest alone takes longer.
inline double attn_wide_us(int nfrag, int n_heads, int causal, int num_cu, int resident, const AtCost& c)
{
    const int owners = c.form.owners, streams = c.form.waves / owners;
    const double blocks = (double)((nfrag + 2 * owners - 1) / (2 * owners)) * n_heads;
    const double chain = (nfrag + streams - 1) / streams, places = (double)num_cu * resident;
    if (causal)
        return c.start + std::fmax(c.block + chain * c.alone, (blocks > 2.0 * places ? c.even : c.pairs) +
                                                                  blocks / num_cu * (c.block / resident + 0.5 * chain * c.shared));
    auto round = [&](double beside) { return beside > 0.0 ? c.block + chain * std::fmax(c.alone, beside * c.shared) : 0.0; };
    const double whole = std::floor(blocks / places);
    return c.start + whole * round(resident) + round(std::ceil((blocks - whole * places) / num_cu));
}

// The narrow pair's workgroups are all resident where it is in question (up to five a compute unit): a unit takes the longest one's
// chain, a memory latency per fragment (`alone`), or the products of all that it holds (`shared` per fragment and half of that per workgroup).  Under the causal mask
// that depends on which fragments meet on a unit: where the fragments of a head divide its turn, one holds nothing but last ones
// (d = 64, 512 tokens x 64 heads 26.4 us, wide 18.7; 700 x 24 18.3 and 21.2 with as many per unit).
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
            load[at] += 2 * f + 9;                                      // (f + 1) / 4 streamed fragments and what 7/8 of one take, in eighths
            most = load[at] > most ? load[at] : most;
            if (++at == units) at = 0;
        }
    return start + std::fmax(chain * alone, most / 8.0 * shared);
}

// Whole score, us, d = 128, narrow / blocks of 128 by eight wavefronts / of 256 / of 128 by four wavefronts, two at a time on a unit:
//                        causal                        unmasked
//     512 x 20   26.1 / 19.3 / 28.1 / 20.8     27.0 / 18.1 / 24.7 / 18.6
//    1000 x  8   26.7 / 27.6 / 42.9 / 31.2     27.3 / 26.6 / 39.9 / 29.6
//    2048 x  8   56.7 / 43.2 / 70.6 / 50.7     68.5 / 41.9 / 67.2 / 48.9
//    4096 x  1   81.8 / 73.6 / 125  / 89.4     83.3 / 72.3 / 123  / 88.0
//     512 x 96   53.4 / 31.2 / 29.9 / 24.6     63.0 / 34.0 / 26.4 / 26.5
//    1400 x 48   133  / 58.1 / 55.0 / 46.7     201  / 94.7 / 99.5 / 82.4
//    1600 x 44   (-)  / 66.1 / 60.8 / 53.6     (-)  / 110  / 111  / 92.2
//    2048 x 24   127  / 47.9 / 71.3 / 53.8     190  / 81.8 / 69.5 / 73.2
//    4096 x 32   550  / 183  / 160  / 166      942  / 320  / 282  / 298
// d = 64, narrow / blocks of 128 by eight wavefronts / by four, three at a time on a unit (256 tokens a block are nowhere the fastest):
//     512 x 20   16.6 / 17.6 / 17.8            16.7 / 16.1 / 15.9
//    1200 x  8   19.9 / 26.7 / 29.7            26.7 / 25.6 / 28.0
//    2048 x  8   31.6 / 35.7 / 40.6            38.6 / 34.4 / 38.9
//    4096 x  1   39.9 / 58.6 / 69.8            41.1 / 57.6 / 67.5
//    1400 x 48   68.8 / 48.7 / 36.8            106  / 74.2 / 55.7
//    4096 x 48   426  / 207  / 153             723  / 340  / 278
inline AtChoice attn_choice(int nfrag, int n_heads, int causal, int head_dim, int num_cu)
{
    const AtChoice none = {0, kAtWaves};
    if (nfrag < 9) return none;         // 64 tokens x 192 heads 14.7 / 19.6, 200 x 64 16.4 / 18.4, 300 x 64 27.6 / 21.7 (d = 128)
    static constexpr AtCost d128[] = {{{2, 8}, 2.04, 9.84, 2.06, 2.06, 12.2, 6.08},
                                      {{4, 8}, 1.68, 10.44, 1.78, 1.78, 37.2, 14.15},
                                      {{2, 4}, 4.08, 7.21, 1.348, 0.973, 21.8, 9.44}};
    static constexpr AtCost d64[] = {{{2, 8}, 4.93, 6.81, 1.515, 1.515, 13.4, 5.21},
                                     {{2, 4}, 5.21, 5.19, 0.967, 0.725, 2.89, 8.07}};
    double best = head_dim == 128 ? attn_narrow_us(nfrag, n_heads, causal, num_cu, 7.34, 2.41, 1.857)
                                  : attn_narrow_us(nfrag, n_heads, causal, num_cu, 7.74, 1.064, 0.908);
    AtChoice choice = none;
    auto consider = [&](const AtCost& c) {
        const double us = attn_wide_us(nfrag, n_heads, causal, num_cu, at_resident(head_dim, c.form.waves), c);
        if (us < best) {
            best = us;
            choice = c.form;
        }
    };
    if (head_dim == 128)
        for (const AtCost& c : d128) consider(c);
    else
        for (const AtCost& c : d64) consider(c);
    return choice;
}

}  // namespace dymoe
