// Which kernels the attention-derived token score takes for a size (attention.hip): host code only.
#pragma once
#include <cmath>
#include <limits>

namespace dymoe {

constexpr int kAtWaves = 4;         // wavefronts of a workgroup of the narrow pair

// Which pair of kernels, by what each is expected to take.  Narrow: a workgroup per 32-token fragment, its wavefronts sharing the streamed
// tokens (many workgroups, operands straight from global memory).  Wide: blocks of 128 or 256 tokens with the stream in LDS, four
// wavefronts sharing a stream or two.  The numbers are those of the whole score in us, fitted to 372 sizes a head size (1 to 64
// heads of 257 to 8000 tokens, both masks; the wide pairs' errors are 4 % rms, the narrow one's 4 to 5 in the range where it matters), so that
// the pair taken is 0.2 % (d = 128) and 0.4 % (d = 64) slower than the best of them on average (with lines drawn at fragment counts alone 1.4 % and 1.3,
// and up to half).
struct AtCost {
    double start;               // launches, score kernel, ends of both passes
    double block;               // a block's own start and end
    double fragment;            // a streamed fragment of a block's chain
    double even;                // causal: what an uneven end adds
};

// Unmasked, all blocks are alike and go over the chip in rounds; causal blocks come longest first and fill it evenly, unless the
// longest alone takes longer.
inline double attn_wide_us(int nfrag, int n_heads, int causal, int num_cu, int owners, const AtCost& c)
{
    const double blocks = (double)((nfrag + 2 * owners - 1) / (2 * owners)) * n_heads;
    const int streams = 8 / owners;
    const double chain = (nfrag + streams - 1) / streams * c.fragment;
    if (!causal) return c.start + std::ceil(blocks / num_cu) * (c.block + chain);
    return c.start + std::fmax(c.block + chain, c.even + blocks / num_cu * (c.block + 0.5 * chain));
}

// The narrow pair's workgroups are all resident where it is in question (up to five a compute unit): a unit takes the longest one's
// chain, a memory latency per fragment (`alone`), or the products of all that it holds (`shared` per fragment).  Under the causal mask
// that depends on which fragments meet on a unit: where the fragments of a head divide its turn, one holds nothing but last ones
// (512 tokens x 64 heads 26.4 us, wide 18.7; 700 x 24 18.3 and 21.2 with as many per unit).
inline double attn_narrow_us(int nfrag, int n_heads, int causal, int num_cu, double start, double alone, double shared)
{
    const long all = (long)nfrag * n_heads;
    if (all > 5L * num_cu) return std::numeric_limits<double>::infinity();
    const int chain = (nfrag + kAtWaves - 1) / kAtWaves;
    if (!causal || all <= num_cu) return start + chain * std::fmax(alone, (double)((all + num_cu - 1) / num_cu) * shared);
    // the narrow kernels' order, one XCD of it where the heads divide: a workgroup a unit in turn
    const bool whole_heads = n_heads % 8 == 0 && num_cu >= 8;
    int load[512] = {}, most = 0;
    const int heads = whole_heads ? n_heads / 8 : n_heads;
    const int units = (whole_heads ? num_cu / 8 : num_cu) < 512 ? (whole_heads ? num_cu / 8 : num_cu) : 512;
    for (int h = 0, at = 0; h < heads; h++)
        for (int f = 0; f < nfrag; f++) {
            load[at] += f / kAtWaves + 1;
            most = load[at] > most ? load[at] : most;
            if (++at == units) at = 0;
        }
    return start + std::fmax(chain * alone, most * shared);
}

// 0: the narrow pair, else tokens per block of the wide pair, in units of 64.  Whole score, us, narrow / 128 / 256 tokens a block:
//                    d = 128, causal          unmasked                 d = 64, causal           unmasked
//     512 x  20   26.1 / 19.3 / 28.2   27.2 / 18.2 / 24.5      16.6 / 17.6 / 25.5   16.7 / 16.1 / 22.0
//    1000 x   8   26.9 / 27.6 / 42.9   27.4 / 26.4 / 39.6      16.3 / 24.0 / 37.5   17.0 / 22.7 / 34.4
//    1200 x   8   33.5 / 31.4 / 48.3   44.8 / 30.6 / 45.3      19.9 / 26.7 / 42.0   26.7 / 25.6 / 38.8
//    2048 x   8   57.0 / 43.0 / 70.0   68.7 / 41.9 / 66.9      31.6 / 35.7 / 60.1   38.6 / 34.4 / 56.9
//    4096 x   1   81.9 / 73.5 / 126    83.5 / 72.4 / 122       39.9 / 58.6 / 106    41.1 / 57.6 / 103
//    1400 x  48  133.6 / 58.1 / 55.1    203 / 96.1 / 99.9      68.8 / 48.7 / 46.6    106 / 74.2 / 81.5
inline int attn_owners(int nfrag, int n_heads, int causal, int head_dim, int num_cu)
{
    if (nfrag < 9) return 0;            // 64 tokens x 192 heads 14.7 / 19.6, 200 x 64 16.4 / 18.4, 300 x 64 27.6 / 21.7 (d = 128)
    const AtCost two = head_dim == 128 ? AtCost{0.4, 10.5, 2.05, 8.2} : AtCost{3.3, 7.7, 1.51, 7.4};
    const AtCost four = head_dim == 128 ? AtCost{0.0, 11.7, 1.85, 15.8} : AtCost{3.6, 7.5, 1.5, 15.0};
    const double narrow = head_dim == 128 ? attn_narrow_us(nfrag, n_heads, causal, num_cu, 8.0, 2.3, 1.9)
                                          : attn_narrow_us(nfrag, n_heads, causal, num_cu, 8.1, 0.97, 0.92);
    const double us2 = attn_wide_us(nfrag, n_heads, causal, num_cu, 2, two), us4 = attn_wide_us(nfrag, n_heads, causal, num_cu, 4, four);
    if (narrow <= std::fmin(us2, us4)) return 0;
    return us2 < us4 ? 2 : 4;
}

}  // namespace dymoe
