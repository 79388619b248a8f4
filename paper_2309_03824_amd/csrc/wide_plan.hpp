// How the columns of a product with a short reduction and a wide result are dealt to workgroups (see mfma_wide.hip).
#pragma once
#include <algorithm>
#include <cstdint>

namespace lrd {

// Chunks of columns per workgroup, of `all`, with `rows` workgroups to each range of columns and `slots` of them at a time: the
// fewest rounds times what a workgroup takes, a chunk and a half of it before its first result leaves.  For each number of rounds
// the shortest ranges that fit it are the candidate, and more rounds than the best cost allows for a single chunk need no look: a few
// steps whatever the width (trying every length took 7 us of the host at 128256 columns).
inline int wide_chunks(int64_t rows, int all, int64_t slots)
{
    int best = all;
    double least = 1e30;
    for (int64_t rounds = (rows + slots - 1) / slots; (double)rounds * 2.5 <= least; ++rounds) {
        const int64_t ranges = std::min<int64_t>(all, rounds * slots / rows);
        const int n = (int)((all + ranges - 1) / ranges);
        const int64_t workgroups = rows * ((all + n - 1) / n);
        const double cost = (double)((workgroups + slots - 1) / slots) * (n + 1.5);
        if (cost <= least) { least = cost; best = n; }
    }
    return best;
}

}  // namespace lrd
