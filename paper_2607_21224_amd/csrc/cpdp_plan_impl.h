// Multi-tensor plan kernels of the local and synchronisation steps and their
// dispatch, generic over where a step's scalars come from (DirectScalars:
// launch arguments; TableScalars: a device step table).  kernels_plan.hip
// and kernels_plan_table.hip instantiate one source each.
#pragma once

#include "cpdp_split.h"

namespace cpdp {
namespace {

// Which search finds a block's tensor in the local step and in the
// thread-per-coordinate synchronisation step.  While every SIMD has at most two
// wavefronts, each block's chain of loads is the time, and one 64-lane load is
// shorter than log2(n) scalar ones from 5 on (30 tensors, 585 blocks: local step
// 2.70 us by the wavefront, 2.87 by the scalar search; synchronisation step of one
// replica 3.82, 3.99) and longer than 2 (4 tensors: 2.65, 2.61; 3.72, 3.69).
// With more blocks they hide each other's chain and the wide loads get in the way
// of the data's (2,490 blocks, 4 tensors, a state that is not in the cache: 4.49,
// 3.92; 6.63, 5.72).  Two kinds of plan keep them up to 6144: one whose large table
// the scalar search waits longer for (600 tensors, 4,700 blocks: 7.2, 8.3; 10.5,
// 11.3; local step of 4 replicas of 120 tensors, 2,260 blocks: 4.71, 5.33), and one
// of 33 to 64 tensors, which one load of 64 lanes and six scalar ones tell apart
// (local step of 4 replicas of 62 tensors, 4,180 blocks: 4.93, 5.19 and, not in the
// cache, 5.85, 5.77; of 2 of 120 tensors 5.37, 5.27 and 6.24, 6.07).  Decided here:
// as a launch argument it cost the host 0.1 us.
// The split step, whose groups all search, is level or faster with the wavefront's.
__device__ __forceinline__ int64_t plan_tensor_by_size(const PlanView& v, int W, int n,
                                                       int64_t b) {
    const bool wide = (int64_t)W * n > 256 || (n > 32 && n <= 64);
    const unsigned most = wide ? 6144 : 2048;
    return n > 8 && gridDim.x <= most ? plan_tensor(v, n, b) : plan_tensor_scalar(v, n, b);
}

// cell (row, chunk b), in the local step's block order -> replica row, tensor t,
// its chunk
template <Opt O, class PS, class Src>
__global__ __launch_bounds__(kBlock) void local_step_plan_kernel(Src src,
                                                                 const int64_t* __restrict__ plan,
                                                                 int W, int n,
                                                                 int64_t total_chunks) {
    const int64_t cell = local_cell(total_chunks * W);
    if (cell < 0) return;
    const PlanView v = plan_view(plan, W, n);
    const int64_t row = cell / total_chunks;
    const int64_t b = cell - row * total_chunks;
    const int64_t t = plan_tensor_by_size(v, W, n, b);
    // the tensor's size and its four addresses come in one round trip: behind
    // the test of p0 the addresses would take a second one
    const int64_t k = row * n + t;
    int64_t P = v.numel[t], start = v.chunk_start[t];
    int64_t prm = v.params[k], m = v.mom[k], m2 = v.mom2[k], g = v.grads[k];
    asm volatile("" : "+s"(P), "+s"(start), "+s"(prm), "+s"(m), "+s"(m2), "+s"(g));
    const int64_t p0 = ((b - start) * kBlock + threadIdx.x) * kVec;
    if (p0 >= P) return;
    local_dispatch<O, PS>(src, global_ptr<typename PS::T>(prm), global_ptr<float>(m),
                          global_ptr<float>(m2), global_ptr<const float>(g), p0, P);
}

// block b -> tensor t and its chunk; run-time W
template <Sync M, Opt O, class PS, bool EXTRA, class Src>
__global__ __launch_bounds__(kBlock) void sync_plan_kernel(Src src,
                                                           const int64_t* __restrict__ plan, int W,
                                                           int n, float inv_w, unsigned flags) {
    const PlanView v = plan_view(plan, W, n);
    const int64_t b = blockIdx.x;
    const int64_t t = plan_tensor_by_size(v, W, n, b);
    const int64_t P = v.numel[t];
    const int64_t p0 = ((b - v.chunk_start[t]) * kBlock + threadIdx.x) * kVec;
    if (p0 >= P) return;
    StepEntry e;
    if (!src.get(e)) return;
    const Table<PS> r{v.params, v.mom, v.mom2, v.grads, n, t};
    float* slow = global_ptr<float>(v.slow[t]);
    float* anchor = global_ptr<float>(v.anchor[t]);
    for_lanes(p0, P, [&](auto lanes, int n) {
        sync_chunk<M, O, 0, PS, lanes, EXTRA>(e.o, r, slow, anchor, W, p0, n, e.beta, e.alpha_lr,
                                              inv_w, flags);
    });
}

// the split step over chunk b's tensor, for every W it takes (AdamW reconcile of
// 4 x 271,117 coordinates in 62 tensors, not in the cache, with the search by 64
// lanes: 13.5 -> 9.1 us; weight decay, 8 x 23.7 M in 161 tensors: 764 -> 695 us,
// 6.0 TB/s).  The thread-per-coordinate band of the flat rows does not hold here:
// on plans it is up to 17 % faster at 1200-2000 chunks and 4-10 % slower just past
// 1024 and 2048 and for AdamW.
template <Sync M, Opt O, int R, class PS, bool EXTRA, class Src>
__global__ __launch_bounds__(kSplitThreads, split_waves(R)) void sync_plan_split_kernel(
    Src src, const int64_t* __restrict__ plan, int W, int n, float inv_w, unsigned flags) {
    extern __shared__ __align__(16) float lds[];
    const PlanView v = plan_view(plan, W, n);
    const int64_t b = blockIdx.x;
    const int64_t t = plan_tensor(v, n, b);
    const Table<PS> r{v.params, v.mom, v.mom2, v.grads, n, t};
    split_dispatch<M, O, R, PS, EXTRA>(src, r, global_ptr<float>(v.slow[t]),
                                       global_ptr<float>(v.anchor[t]), W,
                                       (b - v.chunk_start[t]) * kCoords, v.numel[t], inv_w, flags,
                                       lds);
}

template <Opt O, class Src>
int local_plan_o(Param pt, Src src, const int64_t* plan, int W, int n, int64_t total_chunks,
                 void* stream) {
    const int64_t blocks = local_grid(total_chunks * W);
    return pt == Param::BF16 ? launch(local_step_plan_kernel<O, ParamBF16, Src>, blocks, stream,
                                      src, plan, W, n, total_chunks)
                             : launch(local_step_plan_kernel<O, ParamF32, Src>, blocks, stream,
                                      src, plan, W, n, total_chunks);
}

template <class Src>
int local_plan_any(Opt opt, Param pt, Src src, const int64_t* plan, int W, int n,
                   int64_t total_chunks, void* stream) {
    switch (opt) {
        case Opt::SGD_WD:
            return local_plan_o<Opt::SGD_WD>(pt, src, plan, W, n, total_chunks, stream);
        case Opt::ADAMW:
            return local_plan_o<Opt::ADAMW>(pt, src, plan, W, n, total_chunks, stream);
        default: return local_plan_o<Opt::SGD>(pt, src, plan, W, n, total_chunks, stream);
    }
}

template <Sync M, Opt O, class PS, class Src>
int sync_plan_t(Src src, const int64_t* plan, int W, int n, int64_t total_chunks,
                unsigned flags, void* stream) {
    const float inv_w = 1.0f / (float)W;
    if (can_split(W, total_chunks, kBlock))
        return with_split_r<O, PS>(W, [&](auto R) {
            return flags != 0 ? launch_split(sync_plan_split_kernel<M, O, R, PS, true, Src>,
                                             total_chunks, W, R, stream, src, plan, W, n, inv_w,
                                             flags)
                              : launch_split(sync_plan_split_kernel<M, O, R, PS, false, Src>,
                                             total_chunks, W, R, stream, src, plan, W, n, inv_w,
                                             flags);
        });
    const int resident =
        run_time_waves(step_kind<M, O, PS>(), W, total_chunks * kCoords, RunTime::Plan);
    if (flags != 0)
        return launch_resident(resident, sync_plan_kernel<M, O, PS, true, Src>, total_chunks,
                               stream, src, plan, W, n, inv_w, flags);
    return launch_resident(resident, sync_plan_kernel<M, O, PS, false, Src>, total_chunks,
                           stream, src, plan, W, n, inv_w, flags);
}

template <Sync M, Opt O, class Src>
int sync_plan_p(Param pt, Src src, const int64_t* plan, int W, int n, int64_t total_chunks,
                unsigned flags, void* stream) {
    return pt == Param::BF16
               ? sync_plan_t<M, O, ParamBF16>(src, plan, W, n, total_chunks, flags, stream)
               : sync_plan_t<M, O, ParamF32>(src, plan, W, n, total_chunks, flags, stream);
}

template <Sync M, class Src>
int sync_plan_o(Opt opt, Param pt, Src src, const int64_t* plan, int W, int n,
                int64_t total_chunks, unsigned flags, void* stream) {
    switch (opt) {
        case Opt::SGD_WD:
            return sync_plan_p<M, Opt::SGD_WD>(pt, src, plan, W, n, total_chunks, flags, stream);
        case Opt::ADAMW:
            return sync_plan_p<M, Opt::ADAMW>(pt, src, plan, W, n, total_chunks, flags, stream);
        default:
            return sync_plan_p<M, Opt::SGD>(pt, src, plan, W, n, total_chunks, flags, stream);
    }
}

template <class Src>
int sync_plan_any(Sync mode, Opt opt, Param pt, Src src, const int64_t* plan, int W, int n,
                  int64_t total_chunks, unsigned flags, void* stream) {
    switch (mode) {
        case Sync::LocalSGD:
            return sync_plan_o<Sync::LocalSGD>(opt, pt, src, plan, W, n, total_chunks, flags,
                                               stream);
        case Sync::DDP:
            return sync_plan_o<Sync::DDP>(opt, pt, src, plan, W, n, total_chunks, flags, stream);
        default:
            return sync_plan_o<Sync::CPDP>(opt, pt, src, plan, W, n, total_chunks, flags, stream);
    }
}

}  // namespace
}  // namespace cpdp
