// How the work of a displacement-histogram launch is dealt to blocks (host
// arithmetic, no device code).
//
// A work item is kHistItem particles of one snapshot pair.  A block counts in 32
// bits, at most kHistItem per axis and item, so it takes at most kHistBlockItems
// items: 2^31 counts, whatever bin they fall in.
#pragma once
#include <algorithm>

namespace mdlg {

constexpr int kHistItem = 512;                    // particles of a work item: the threads of a block
constexpr long long kHistBlockItems = 1LL << 22;  // items of one block at most
constexpr int kHistTargetBlocks = 512;            // blocks of a launch aimed at: two per compute unit

// shares[r]: blocks of replica r for each of n_lag lags, where it has items[r]
// items; every replica of the launch gets what the largest one needs.
inline void hist_deal(int n_rep, const long long* items, int n_lag, long long* shares) {
    long long most = 0;
    for (int r = 0; r < n_rep; ++r) most = std::max(most, items[r]);
    const long long target = kHistTargetBlocks / ((long long)n_rep * n_lag);
    const long long least = (most + kHistBlockItems - 1) / kHistBlockItems;
    for (int r = 0; r < n_rep; ++r) shares[r] = std::max({1LL, least, std::min(target, most)});
}

}  // namespace mdlg
