// How the factorisation's tiles and the sweep's columns (gptq.hip) are divided over launches and workgroups: host code only.
#pragma once
#include <initializer_list>

namespace dymoe {

// Tiles (pairs of block rows x pairs of block columns) of panel q: `near` of the pairs q + 1 and q + 2 and `first` of the
// others in the first launch, `later` in the second.  single: half tiles that the second launch brings forward by one step.
// A launch's tiles are taken by halves (a block row each).
struct GqWide {
    long q, pairs, near, first, later, single;
};
// Blocks that a worker takes before those behind the solvers start.
constexpr int kGqSkip = 3;
// Workgroups for the tiles: `early` on the compute units that the solvers leave, or, from as many solvers as units on, that have one solver less
// than the others (17408 columns, 272 solvers on 256 units: 45.3 ms with every worker the same share, 43.6 so, 43.9 with three small workgroups
// on a unit); where these would take longer than kGqSkip blocks each, one behind each other solver as well.
inline long gq_early(long nb, long num_cu) { return num_cu - nb % num_cu; }
inline long gq_workers(long nb, long num_cu, long blocks)
{
    const long early = gq_early(nb, num_cu);
    return blocks <= kGqSkip * early ? (blocks < early ? blocks : early) : num_cu;
}
// How long a launch takes, in blocks of the worker with the most of them (5 us each): the solver's chain is 2.7 of them, a worker's start half of one.
inline double gq_launch_length(long nb, long num_cu, long blocks)
{
    const long early = gq_early(nb, num_cu);
    const long rounds = blocks <= kGqSkip * early ? (blocks + early - 1) / (early > 0 ? early : 1)
                                                  : kGqSkip + (blocks - kGqSkip * early + num_cu - 1) / num_cu;
    return rounds + 0.5 > 2.7 ? rounds + 0.5 : 2.7;
}
// The tiles of panel q's two launches, whose blocks are `fixed` + 2 first and `all` less those: the split for which both together take
// the fewest rounds, of those the most even one.  (In equal halves each launch's last round is half empty on average: K = 8192 5614 us, so
// 5474; 4096 1139 and 1112.)
inline long gq_split(long nb, long num_cu, long fixed, long rest, long all)
{
    const long early = gq_early(nb, num_cu), even = (all / 2 - fixed) / 2;
    auto inside = [&](long first) { return first < 0 ? 0 : first > rest ? rest : first; };
    auto length = [&](long first) { return gq_launch_length(nb, num_cu, fixed + 2 * first) + gq_launch_length(nb, num_cu, all - fixed - 2 * first); };
    long best = inside(even);
    double least = length(best);
    // launches that end with a whole round: the first with r of them, or the second
    const long middle = all / 2 <= kGqSkip * early ? all / 2 / (early > 0 ? early : 1) : kGqSkip + (all / 2 - kGqSkip * early) / num_cu;
    for (long r = middle > 3 ? middle - 3 : 1; r <= middle + 3; r++) {
        const long full = r <= kGqSkip ? r * early : kGqSkip * early + (r - kGqSkip) * num_cu;
        for (const long first : {inside((full - fixed) / 2), inside((all - full - fixed + 1) / 2)}) {
            const double len = length(first);
            const long off = first > even ? first - even : even - first, best_off = best > even ? best - even : even - best;
            if (len < least || (len == least && off < best_off)) {
                least = len;
                best = first;
            }
        }
    }
    return best;
}
inline GqWide gq_wide(long nb, long k, long num_cu)
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
        const long fixed = 2 * w.near - 1 - (w.q + 1), single = nb - (2 * w.q + 4) + w.q + 2;      // (the other launch's if k is even)
        w.first = gq_split(nb, num_cu, fixed, rest, fixed + 2 * rest + single);
        w.later = rest - w.first;
    }
    if (k & 1) w.single = nb - (k + 1) + w.q + 2;                   // block column k + 1 from the diagonal down, block row k + 1
    return w;
}
inline long gq_wide_blocks(const GqWide& w, long k)
{
    if (k & 1) return w.single + 2 * w.later;
    return w.near ? 2 * (w.near + w.first) - 1 - (w.q + 1) : 0;     // without the halves in block row k
}

// The sweep: workgroups for the columns [next, K) behind the panel that begins at `base`, which lose the errors of the panel before (the first
// panel has none).  128 rows x 128 columns each from three quarters of one per compute unit on, else 64 x 64.
struct GqBehindGrid {
    bool small;
    long workgroups;
};
inline GqBehindGrid gq_behind_grid(long N, long K, long base, long next, long num_cu)
{
    const long blocks = (N + 63) / 64, row_pairs = (blocks + 1) / 2, col_pairs = (K - next + 127) / 128;
    const bool small = 4 * row_pairs * col_pairs <= 3 * num_cu;
    if (base == 0 || next >= K) return {small, 0};
    return {small, small ? blocks * ((K - next) / 64) : 8 * ((row_pairs + 7) / 8) * col_pairs};
}

}  // namespace dymoe
