// Checks the dispatch of the synchronisation steps (cpdp_dispatch.h) over
// replica counts and sizes: whatever kernel a step goes to, its launch fits.
// Exits non-zero on the first mismatch.
#include <cstdio>
#include <initializer_list>

#include "cpdp_dispatch.h"

static int failures = 0;
#define CHECK(cond, W, P)                                                          \
    do {                                                                           \
        if (!(cond)) {                                                             \
            std::printf("FAIL line %d: W %d P %lld: %s\n", __LINE__, (int)(W),     \
                        (long long)(P), #cond);                                    \
            ++failures;                                                            \
        }                                                                          \
    } while (0)

int main() {
    using namespace cpdp;
    CHECK(launch_fits(0xFFFFFFFF / 64, 64), 0, 0);
    CHECK(!launch_fits(((int64_t)1 << 32) / 64, 64), 0, 0);

    for (int group : {64, 256}) {
        const int64_t per_block = (int64_t)group * 4;
        auto blocks = [&](int64_t P) { return (P + per_block - 1) / per_block; };
        for (int W = 1; W <= 40; ++W)
            for (int e = 0; e <= 34; ++e)
                for (int64_t d : {-1, 0, 1}) {
                    const int64_t P = ((int64_t)1 << e) + d;
                    if (P < 1) continue;
                    const bool split = can_split(W, blocks(P), group);
                    for (int R : {1, 2, 4}) {
                        const int64_t threads = split_threads(W, R, group);
                        if (split && threads <= kSplitThreads)
                            CHECK(launch_fits(blocks(P), threads), W, P);
                    }
                    // sizes that fit stay with the split step
                    if (W >= kSplitMinW && W <= split_max_w(group) && P <= ((int64_t)1 << 29))
                        CHECK(split, W, P);
                    if (W < kSplitMinW || W > split_max_w(group)) CHECK(!split, W, P);
                }
    }
    // states of about 120 to 215 GB on one GPU: 16 replicas of 2^30 coordinates
    // and 8 of 2^31 have one thread too many for the split step, and fit the
    // one-wavefront blocks of the thread-per-coordinate kernel
    CHECK(!can_split(16, ((int64_t)1 << 30) / 256, 64), 16, (int64_t)1 << 30);
    CHECK(!can_split(8, ((int64_t)1 << 31) / 256, 64), 8, (int64_t)1 << 31);
    CHECK(can_split(16, ((int64_t)1 << 30) / 256 - 1, 64), 16, (int64_t)1 << 30);
    CHECK(launch_fits(((int64_t)1 << 30) / 256, 64), 16, (int64_t)1 << 30);
    CHECK(launch_fits(((int64_t)1 << 31) / 256, 64), 8, (int64_t)1 << 31);
    // the rules between the two kernels: what has nothing to split is never
    // weighed, sizes far on either side go to the split step whatever the types
    // are, and every line is a single one (no gaps between a kernel's sizes
    // other than where whole vectors end)
    for (Sync m : {Sync::CPDP, Sync::LocalSGD, Sync::DDP})
        for (Opt o : {Opt::SGD, Opt::SGD_WD, Opt::ADAMW})
            for (int types = 0; types < 8; ++types)
                for (int W = kSplitMinW; W <= 32; ++W) {
                    const StepKind k{m, o, (types & 1) != 0, (types & 2) != 0, (types & 4) != 0};
                    const bool none = column_last(k, W) == INT64_MAX;
                    const bool many = (types & 3) == 3 && W > (m == Sync::CPDP ? 8 : 16);
                    const bool wide = types >= 6 && m == Sync::CPDP && W > 16 && W <= 30;
                    CHECK(none == (many || wide), W, types);
                    int turns = 0;
                    bool before = false;
                    for (int64_t waves = 1; waves < 20000; ++waves) {
                        const bool column = takes_columns(k, W, waves * 256 - 1, true);
                        if (column) {
                            CHECK(waves >= 640 && W * waves > 8192, W, waves);
                            CHECK(none || waves <= 8192, W, waves);
                        }
                        turns += column != before;
                        before = column;
                        // ragged rows of a compile-time-W kernel: from a wavefront a SIMD on
                        if (waves < 640) CHECK(!takes_columns(k, W, waves * 256 - 1, false), W, waves);
                        if (o == Opt::ADAMW)
                            CHECK(takes_columns(k, W, waves * 256, true) ==
                                      takes_columns(k, W, waves * 256, false), W, waves);
                    }
                    CHECK(turns <= 2, W, turns);
                    if (!none) CHECK(!takes_columns(k, W, (int64_t)1 << 33, false), W, types);
                    CHECK(ddp_mean_waves(k, W, 1 << 20, true) == 0 || W > 8, W, types);
                    CHECK(ddp_mean_waves(k, W, 1 << 23, false) == 0, W, types);
                    CHECK((ddp_mean_waves(k, W, 1 << 23, true) != 0) ==
                              (m == Sync::DDP && W <= 6), W, types);
                    if (o == Opt::ADAMW) CHECK(!fixed_w(k, W), W, types);
                    // rows of whole vectors only, and never the ragged ones beside them
                    CHECK(takes_columns({Sync::CPDP, Opt::SGD, false, false}, 8, 4096, false), 8, 4096);
                    CHECK(!takes_columns({Sync::CPDP, Opt::SGD, false, false}, 8, 4097, false), 8, 4097);
                }
    // wavefronts of the run-time-W kernel: large states of one and two replicas only
    const StepKind sgd{Sync::CPDP, Opt::SGD, false, false}, adam{Sync::CPDP, Opt::ADAMW, false, false};
    const StepKind ddp{Sync::DDP, Opt::SGD, false, false};
    for (RunTime r : {RunTime::Table, RunTime::Plan, RunTime::Variant})
        for (int W = 1; W <= 40; ++W) {
            const int64_t large = ((int64_t)1 << 24) / W;
            const bool plan = r == RunTime::Plan, few = W <= 2;
            CHECK(run_time_waves(sgd, W, large - 1, r) == 0, W, large - 1);
            CHECK(run_time_waves(sgd, W, large, r) == (!few ? 0 : plan && W == 1 ? 5 : 3), W, large);
            CHECK(run_time_waves(adam, W, large, r) == (few && r == RunTime::Table ? 3 : 0), W, large);
            CHECK(run_time_waves(ddp, W, large, r) == (!few ? 0 : plan ? 6 : W == 2 ? 3 : 0), W, large);
        }
    std::printf("%s\n", failures ? "FAILED" : "OK");
    return failures ? 1 : 0;
}
