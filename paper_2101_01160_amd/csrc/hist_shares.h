// How the work of a displacement-histogram launch is dealt to blocks (host
// arithmetic, no device code).
//
// A work item is kHistItem particles of one snapshot pair.  A block counts in 32
// bits, at most kHistItem per axis and item, so it takes at most kHistBlockItems
// items: 2^31 counts, whatever bin they fall in.
#pragma once
#include <algorithm>

namespace mdlg {

constexpr int kHistItem = 512;                    // particles of a work item at most: the threads of a block
constexpr long long kHistBlockItems = 1LL << 22;  // items of one block at most
constexpr int kHistTargetBlocks = 512;            // blocks of kHistItem threads aimed at: two per compute unit

// shares[r]: blocks of replica r for each of n_lag lags, where it has items[r]
// items: its part of the blocks aimed at, by its items.  (With as many for each
// replica, 16 blocks were left for the large one of 2^20 particles among 31 of
// 4096: 522 us for 9 snapshots and one lag, 18.3 ms for 20 and 16 lags.)
// Blocks of fewer threads are as many more.
inline void hist_deal(int n_rep, const long long* items, int n_lag, long long* shares, int threads = kHistItem) {
    long long total = 0;
    for (int r = 0; r < n_rep; ++r) total += items[r];
    const double scale = total > 0 ? std::max(1, kHistTargetBlocks * (kHistItem / threads) / n_lag) / (double)total : 0.0;
    for (int r = 0; r < n_rep; ++r) {
        const long long part = (long long)((double)items[r] * scale);
        const long long least = (items[r] + kHistBlockItems - 1) / kHistBlockItems;  // 0 without items
        shares[r] = std::max(least, std::min(part, items[r]));
    }
}

}  // namespace mdlg
