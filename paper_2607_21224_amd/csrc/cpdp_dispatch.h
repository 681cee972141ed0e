// Which kernel takes a synchronisation step, as plain host arithmetic on sizes
// (no HIP), so that a host-only program can check it for every size.
#pragma once
#include <stdint.h>

namespace cpdp {

// A launch may hold fewer than 2^32 work items in a dimension; HIP refuses a
// larger one.
constexpr bool launch_fits(int64_t blocks, int64_t threads) {
    return blocks <= (int64_t)0xFFFFFFFF / threads;
}

// Threads of a block of the split step at most: 16 groups of one wavefront.
// With 8 groups (two replicas a group at W = 16) the reconcile of 16 x 23.9 M
// fp32 coordinates took 1433 us instead of 1361, with 4 groups (four replicas
// each) 1431.
constexpr int kSplitThreads = 1024;

// Replicas the split step takes: at W = 1 and 2 there is nothing to split (the
// thread-per-coordinate kernel is up to 0.4 us faster on small states and
// level on large ones); 32 are two rows a group of 16 and 32 KB of LDS.
constexpr int kSplitMinW = 3;
constexpr int split_max_w(int group) { return 2 * (kSplitThreads / group); }

// Threads of a split block whose groups of `group` threads hold R replicas
constexpr int64_t split_threads(int W, int R, int group) {
    return (int64_t)((W + R - 1) / R) * group;
}

// Whether the split step can take W replicas in `blocks` blocks.  A group holds
// one replica up to 16 groups, and more above, so a launch never has more
// threads than with one replica a group, 16 groups at most.
constexpr bool can_split(int W, int64_t blocks, int group) {
    return W >= kSplitMinW && W <= split_max_w(group) &&
           launch_fits(blocks, W * group < kSplitThreads ? W * group : kSplitThreads);
}

}  // namespace cpdp
