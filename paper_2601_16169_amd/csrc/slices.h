// Host side of the sliced tables: the order of the rows, how many lanes a long
// row takes and which wave of a workgroup walks which slice.
#pragma once

#include <algorithm>
#include <vector>

#include "sqd_internal.h"

// Rows by decreasing length (ties by index): a counting sort.
inline std::vector<int> rows_longest_first(const std::vector<int>& len) {
    const int most = len.empty() ? 0 : *std::max_element(len.begin(), len.end());
    std::vector<int> at(most + 2, 0), rows(len.size());
    for (int l : len) at[most - l + 1] += 1;
    for (int k = 0; k <= most; ++k) at[k + 1] += at[k];
    for (size_t r = 0; r < len.size(); ++r) rows[at[most - len[r]]++] = (int)r;
    return rows;
}

// Lanes per row (log2): the fewest that keep a lane's entries at or below cap.
inline int split_of(int len, int cap) {
    int k = 0;
    while (k < 6 && ((len + (1 << k) - 1) >> k) > cap) ++k;
    return k;
}

// Slices dealt into bins, the costliest into the lightest bin; the heaviest
// bins are placed beside the lightest, so that pairs and fours of adjacent
// bins are even too.
inline std::vector<std::vector<int>> deal_bins(const std::vector<int>& cost) {
    std::vector<int> order(cost.size()), load(kBins, 0), rank(kBins);
    for (size_t k = 0; k < order.size(); ++k) order[k] = (int)k;
    std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return cost[x] > cost[y]; });
    std::vector<std::vector<int>> in(kBins), out(kBins);
    for (int k : order) {
        const int q = (int)(std::min_element(load.begin(), load.end()) - load.begin());
        in[q].push_back(k);
        load[q] += cost[k];
    }
    for (int q = 0; q < kBins; ++q) rank[q] = q;
    std::stable_sort(rank.begin(), rank.end(), [&](int x, int y) { return load[x] > load[y]; });
    static constexpr int kPlace[kBins] = {0, 15, 7, 8, 3, 12, 4, 11, 1, 14, 6, 9, 2, 13, 5, 10};
    for (int q = 0; q < kBins; ++q) out[q] = in[rank[kPlace[q]]];
    return out;
}

// Entries a lane of a table with split rows takes at most.  A wavefront walks
// a slice at the pace of its longest lane, and the rows of sampled sets are
// uneven: the Hartree-Fock string reaches half of the set, the mean row a
// tenth.  A thirty-second of all columns leaves each of sixteen waves about
// two slices of that length, so the waves of a workgroup end together, and
// only the long rows pay for the sums across lanes.
inline int split_cap(int64_t entries, int least) { return (int)std::max<int64_t>(least, (entries + 2047) / 2048); }
