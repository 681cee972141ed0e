// The flat-layout synchronisation kernels (CPDP reconcile, LocalSGD averaging,
// DDP gradient step) and their dispatch over update rule, parameter,
// gradient and momentum storage types, and W.  Each strategy is instantiated in
// a translation unit of its own (kernels_sync_<strategy>.hip) so the three
// compile in parallel.
#pragma once

#include "cpdp_device.h"
#include "cpdp_split.h"

namespace cpdp {
namespace {

// WT: replicas at compile time; 0: at run time; kManyW: at run time, more than the
// split step takes.  AdamW's long update on that many replicas is faster with two
// wavefronts a SIMD that keep more of a batch in registers than with four (40 x
// 100,000 fp32 coordinates: 37.7 us with four, 33.9 with two; 3.0 M level).
constexpr int kManyW = -1;
constexpr int column_waves_max(Opt O, int WT) { return O == Opt::ADAMW && WT == kManyW ? 2 : 8; }

template <Sync M, Opt O, int WT, class PS, bool EXTRA, class GS, class MS>
__global__ __launch_bounds__(kBlock)
__attribute__((amdgpu_waves_per_eu(1, column_waves_max(O, WT)))) void sync_kernel(
    OptParams o, typename PS::T* __restrict__ params, typename MS::T* __restrict__ mom,
    float* __restrict__ mom2, GradPtr<EXTRA, GS> __restrict__ grads, float* __restrict__ slow,
    float* __restrict__ anchor, int W, int64_t ld, int64_t P, float beta, float alpha_lr,
    float inv_w, unsigned flags) {
    const int64_t p0 = ((int64_t)blockIdx.x * kBlock + threadIdx.x) * kVec;
    if (p0 >= P) return;
    // Strided holds mutable row pointers; without EXTRA no store to the
    // gradient rows is instantiated
    const Strided<PS, GS, MS> r{params, mom, mom2, const_cast<typename GS::T*>(grads), ld};
    for_lanes(p0, P, [&](auto lanes, int n) {
        sync_chunk<M, O, WT, PS, lanes, EXTRA>(o, r, slow, anchor, W, p0, n, beta, alpha_lr, inv_w,
                                               flags);
    });
}

template <Sync M, Opt O, int WT, class PS, bool EXTRA = false, class GS = ParamF32,
          class MS = ParamF32>
int sync_w(const OptParams& o, const SyncArgs& a, int resident = 0) {
    using T = typename PS::T;
    const float alpha_lr = a.alpha * o.lr;
    const float inv_w = 1.0f / (float)a.W;
    // the variants run only from the entry points whose gradient argument is
    // mutable (flags != 0), so dropping const here restores the caller's type
    const GradPtr<EXTRA, GS> grads =
        const_cast<typename GS::T*>(static_cast<const typename GS::T*>(a.grads));
    return launch_resident(resident, sync_kernel<M, O, WT, PS, EXTRA, GS, MS>, blocks_for(a.P),
                           a.stream, o, static_cast<T*>(a.params),
                           static_cast<typename MS::T*>(a.mom), a.mom2, grads, a.slow, a.anchor,
                           a.W, a.ld, a.P, a.beta, alpha_lr, inv_w, a.flags);
}

// Which kernel takes the step (the rules and what they were measured at are in
// cpdp_dispatch.h).
template <Sync M, Opt O, class PS, class GS = ParamF32, class MS = ParamF32>
int sync_t(const OptParams& o, const SyncArgs& a) {
    constexpr StepKind kind = step_kind<M, O, PS, GS, MS>();
    const int mean_waves = ddp_mean_waves(kind, a.W, a.P, a.flags & kSyncWriteGbar);
    const bool split = can_split(a.W, blocks_for(a.P), kBlock) && mean_waves == 0 &&
                       !takes_columns(kind, a.W, a.P, a.flags != 0);
    const DirectScalars src{o, a.beta, a.alpha * o.lr};
    if constexpr (std::is_same<GS, ParamF32>::value && std::is_same<MS, ParamF32>::value) {
        if (a.flags != 0) {
            const int resident =
                mean_waves != 0 ? mean_waves : run_time_waves(kind, a.W, a.P, RunTime::Variant);
            return split ? sync_split<M, O, PS, true, GS, MS>(src, a)
                         : sync_w<M, O, 0, PS, true>(o, a, resident);
        }
    }
    if (split) return sync_split<M, O, PS, false, GS, MS>(src, a);
    if (a.W == 1) return sync_w<M, O, 1, PS, false, GS, MS>(o, a);
    if (a.W == 2) return sync_w<M, O, 2, PS, false, GS, MS>(o, a);
    if constexpr (fixed_w(kind, 4))
        if (a.W == 4) return sync_w<M, O, 4, PS, false, GS, MS>(o, a);
    if constexpr (fixed_w(kind, 8)) {
        if (a.W == 8) return sync_w<M, O, 8, PS, false, GS, MS>(o, a);
        if (a.W == 16) return sync_w<M, O, 16, PS, false, GS, MS>(o, a);
    }
    if constexpr (O == Opt::ADAMW)
        if (a.W > split_max_w(kBlock)) return sync_w<M, O, kManyW, PS, false, GS, MS>(o, a);
    return sync_w<M, O, 0, PS, false, GS, MS>(o, a);
}

// bf16 gradients or momentum: momentum SGD without variants only (the
// validation layer enforces it)
template <Sync M, class PS>
int sync_narrow(Grad gt, Mom mt, const OptParams& o, const SyncArgs& a) {
    if (a.flags != 0) return (int)hipErrorInvalidValue;
    if (gt == Grad::BF16)
        return mt == Mom::BF16 ? sync_t<M, Opt::SGD, PS, ParamBF16, ParamBF16>(o, a)
                               : sync_t<M, Opt::SGD, PS, ParamBF16, ParamF32>(o, a);
    return sync_t<M, Opt::SGD, PS, ParamF32, ParamBF16>(o, a);
}

template <Sync M, Opt O>
int sync_p(Param pt, Grad gt, Mom mt, const OptParams& o, const SyncArgs& a) {
    if (gt == Grad::BF16 || mt == Mom::BF16) {
        if constexpr (O == Opt::SGD)
            return pt == Param::BF16 ? sync_narrow<M, ParamBF16>(gt, mt, o, a)
                                     : sync_narrow<M, ParamF32>(gt, mt, o, a);
        return (int)hipErrorInvalidValue;
    }
    return pt == Param::BF16 ? sync_t<M, O, ParamBF16>(o, a) : sync_t<M, O, ParamF32>(o, a);
}

template <Sync M>
int sync_o(Opt opt, Param pt, Grad gt, Mom mt, const OptParams& o, const SyncArgs& a) {
    switch (opt) {
        case Opt::SGD_WD: return sync_p<M, Opt::SGD_WD>(pt, gt, mt, o, a);
        case Opt::ADAMW: return sync_p<M, Opt::ADAMW>(pt, gt, mt, o, a);
        default: return sync_p<M, Opt::SGD>(pt, gt, mt, o, a);
    }
}

}  // namespace

template <Sync M>
int launch_sync_mode(Opt opt, const OptParams& o, Param pt, Grad gt, Mom mt, void* params,
                     void* mom, float* mom2, const void* grads, float* slow, float* anchor,
                     int W, int64_t P, int64_t ld, float beta, float alpha, unsigned flags,
                     void* stream) {
    const SyncArgs a{params, mom, mom2, grads, slow, anchor, W, P, ld, beta, alpha, flags, stream};
    return sync_o<M>(opt, pt, gt, mt, o, a);
}

}  // namespace cpdp
