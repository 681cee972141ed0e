// Which kernel takes a synchronisation step, as plain host arithmetic on sizes
// (no HIP), so that a host-only program can check it for every size.
#pragma once
#include <stdint.h>

#include "cpdp_launch.h"

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

// A synchronisation step as the rules below see it.
struct StepKind {
    Sync mode;
    Opt opt;
    bool bf16_params, bf16_mom;
    bool bf16_grads = false;
};

// Wavefronts of the thread-per-coordinate kernel (64 threads of 4 coordinates).
constexpr int64_t column_waves(int64_t P) { return (P + 255) / 256; }

// Where the thread-per-coordinate kernel is the faster of the two on three and
// more replicas.  The card holds 8192 wavefronts, 8 on each of 1024 SIMDs.  Up to
// about one round of the split step's W wavefronts per 256 coordinates, its
// single trip to memory wins, and past some four rounds the order of its accesses
// does.  In between, its blocks load and store in step and the last round is
// partly empty, while the other kernel, from somewhat less than a wavefront a SIMD
// to about three, has all of its wavefronts resident at once.  It does not matter
// whether the rows stay in the last-level cache from one call to the next: the
// lines hold for a state that is stepped repeatedly and for states rotated past
// the cache.  Split and thread-per-coordinate, us, rotated:
//   fp32 SGD       6 x 685,068 18.6, 17.3   12 x 342,532 18.8, 17.2
//                  32 x 256,900 34.8, 27.4  12 x 174,763 10.3, 11.0
//                  32 x 786,840 93.2, 102   16 x 1,048,577 62.5, 64.6
//   fp32 AdamW     32 x 287,000 47.5, 42.9  8 x 351,973 16.2, 17.6
//   bf16 params    16 x 513,800 30.3, 25.2  32 x 2,034,000 201, 235
//   all bf16       32 x 1,000,000 83, 63    24 x 1,370,136 103, 72
// Time does not grow evenly there: a kernel is fastest where its wavefronts are a
// multiple of 1024, and a line between two such sizes can be off by 5 %.

// Wavefronts from which, and more than how many of the split step's (AdamW's long
// update hides more of a trip, an all-bf16 row has half the bytes).
constexpr int64_t column_first(const StepKind& k) {
    if (k.opt == Opt::ADAMW) return 1024;
    return k.bf16_params || k.bf16_mom || k.mode == Sync::DDP ? 768 : 640;
}
constexpr int64_t split_round(const StepKind& k, int W) {
    const bool all_bf16 = k.bf16_params && k.bf16_mom;
    if (all_bf16 && k.mode != Sync::CPDP) return 3 * 8192;
    return all_bf16 || (k.opt == Opt::ADAMW && W > 3) ? 8192 + 4096 : 8192;
}
// Wavefronts up to which.  With half the bytes a row the split step gains less and
// the line lies higher; bf16 parameters and momentum on many replicas have none (us,
// split, thread-per-coordinate: 25 x 12.0 M all-bf16 DDP 700, 595; 32 x 40.0 M
// 2621, 2532; LocalSGD 2763, 2540), and neither has a CPDP step whose parameters
// alone are fp32, on 17 to 30 replicas (28 x 2.6 M 231, 201; 28 x 12.0 M 1027, 960,
// but 24 x 12.0 M 811, 830).
constexpr int64_t column_last(const StepKind& k, int W) {
    const bool cpdp = k.mode == Sync::CPDP;
    if (k.bf16_params && k.bf16_mom && W > (cpdp ? 8 : 16)) return INT64_MAX;
    if (cpdp && k.bf16_grads && k.bf16_mom && W > 16 && W <= 30) return INT64_MAX;
    if (k.opt != Opt::ADAMW && k.bf16_mom && W > 16) return 8192;
    if (k.opt != Opt::ADAMW && (k.bf16_params || k.bf16_mom)) return 5120;
    return W < 4 ? 5120 : W <= 12 ? 3328 : 3072;
}
constexpr bool column_band(const StepKind& k, int W, int64_t waves) {
    if (k.bf16_params && k.bf16_mom && W < 4) return false;
    return waves >= column_first(k) && waves <= column_last(k, W) &&
           W * waves > split_round(k, W);
}

// Replica counts of the thread-per-coordinate kernel with W at compile time: all
// loads of a step in flight at once.  Not for AdamW above 2 and bf16 rows above
// 4, where the split step or the run-time-W kernel is faster at every size.
constexpr bool fixed_w(const StepKind& k, int W) {
    if (W == 1 || W == 2) return true;
    if (k.opt == Opt::ADAMW) return false;
    return W == 4 || ((W == 8 || W == 16) && !k.bf16_params && !k.bf16_mom);
}

// Wavefronts up to which the compile-time-W kernel is faster than the split step
// on rows of whole vectors: no LDS, no barriers (fp32 CPDP, 4 x 1,020: 2.3 us
// against 3.0, 8 x 4,092: 2.6 against 3.1, 16 x 4,092: 3.5 against 3.7).  On
// ragged rows the split step is level on 4 replicas and faster on more.
constexpr int64_t fixed_small(const StepKind& k, int W) {
    const bool cpdp = k.mode == Sync::CPDP;
    if (W == 4) return k.bf16_mom && !cpdp ? 0 : 1023;
    if (W == 8) return k.mode == Sync::DDP ? 8 : 1023;
    return W == 16 && cpdp ? 64 : 0;
}
// The same from a wavefront a SIMD on, ragged or not (fp32 CPDP, 4 x 524,289:
// 10.0 us against 10.5, 8 x 262,144: 9.1 against 9.9).
constexpr int64_t fixed_last(const StepKind& k, int W) {
    if (k.bf16_mom && k.mode != Sync::CPDP) return 0;
    return W == 4 ? 5120 : W == 8 ? 4096 : 3072;
}

// Whether a step that could be split goes to the thread-per-coordinate kernel.
// run_time: the variants and the step tables, which have no compile-time W; with
// it the tiniest states of 4 replicas are still 8-17 % faster.
constexpr bool takes_columns(const StepKind& k, int W, int64_t P, bool run_time) {
    const int64_t waves = column_waves(P);
    if (column_band(k, W, waves)) return true;
    const bool whole = P % 4 == 0;
    if (run_time) return W == 4 && k.opt != Opt::ADAMW && whole && waves <= 16;
    if (!fixed_w(k, W) || W < kSplitMinW) return false;
    return (waves >= 1024 && waves <= fixed_last(k, W)) ||
           (whole && waves <= fixed_small(k, W));
}

// A DDP step that writes the gradient mean back streams as many rows out as in.
// Past the cache, on up to 6 replicas, it goes to the thread-per-coordinate kernel
// with two wavefronts a SIMD resident (three on 3 replicas), fewer than fit: the
// memory takes fewer streams better there (6 x 11,173,963: split 297 us, the other
// kernel with the six a SIMD that fit 292, with two 273; 3 x 23.7 M split 280, six
// 291, three 272).  0: the step does not go there.
constexpr int ddp_mean_waves(const StepKind& k, int W, int64_t P, bool writes_mean) {
    if (k.mode != Sync::DDP || !writes_mean || W < kSplitMinW || W > 6) return 0;
    return P < ((int64_t)1 << 23) / W ? 0 : W == 3 ? 3 : 2;
}

// Wavefronts a SIMD that the run-time-W kernel keeps resident on one and two
// replicas (0: as many as fit).  It has room for six, which small and mid-sized
// states are faster with (step table, 2 x 1,141,054 DDP: 9.3 us, 10.5 with three)
// and large ones slower (2 x 16.9 M CPDP 157 and 149, 2 x 15.1 M LocalSGD 110 and
// 106).  DDP on one replica, three rows in all, keeps the six (19.7 M: 63 and 69).
// AdamW keeps as many as fit in plans and variants (plan, 1 x 30 M DDP: 133 us, 141
// when its registers left room for fewer).
// A plan's kernel has room for eight (LocalSGD six) and is best with three only on
// two replicas that are averaged (us with all, three: CPDP 2 x 18.0 M 167, 161;
// 1 x 30 M 179, 181, with five 173; LocalSGD 2 x 20.0 M 148, 140; 1 x 40 M 152,
// 169, with five 154; DDP 2 x 20.0 M 133, 132, with six 129).
enum class RunTime { Table, Plan, Variant };
constexpr int run_time_waves(const StepKind& k, int W, int64_t P, RunTime kernel) {
    if (W >= kSplitMinW || P < ((int64_t)1 << 24) / W) return 0;
    if (k.opt == Opt::ADAMW && kernel != RunTime::Table) return 0;
    if (kernel == RunTime::Plan && k.mode == Sync::DDP) return 6;
    if (kernel == RunTime::Plan && W == 1) return 5;
    return k.mode == Sync::DDP && W == 1 ? 0 : 3;
}

}  // namespace cpdp
