// The flat-layout synchronisation kernels (CPDP reconcile, LocalSGD averaging,
// DDP gradient step) and their dispatch over update rule, parameter,
// gradient and momentum storage types, and W.  Each strategy is instantiated in a translation unit of its own
// (kernels_sync_<strategy>.hip) so the three compile in parallel.
#pragma once

#include "cpdp_device.h"
#include "cpdp_split.h"

namespace cpdp {
namespace {

template <Sync M, Opt O, int WT, class PS, bool EXTRA, class GS, class MS>
__global__ __launch_bounds__(kBlock) void sync_kernel(
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
int sync_w(const OptParams& o, const SyncArgs& a) {
    using T = typename PS::T;
    const float alpha_lr = a.alpha * o.lr;
    const float inv_w = 1.0f / (float)a.W;
    // the variants run only from the entry points whose gradient argument is
    // mutable (flags != 0), so dropping const here restores the caller's type
    const GradPtr<EXTRA, GS> grads =
        const_cast<typename GS::T*>(static_cast<const typename GS::T*>(a.grads));
    return launch(sync_kernel<M, O, WT, PS, EXTRA, GS, MS>, blocks_for(a.P), a.stream, o,
                  static_cast<T*>(a.params), static_cast<typename MS::T*>(a.mom), a.mom2, grads,
                  a.slow, a.anchor, a.W, a.ld, a.P, a.beta, alpha_lr, inv_w, a.flags);
}

// Which kernel takes the step.  The split one, except
//  * W outside its range (W = 1 and 2, and more than 32 replicas), or so many
//    coordinates that its blocks of up to 1024 threads pass the 2^32 work items
//    of a launch (W * P >= 2^34 up to 16 replicas);
//  * fp32 momentum SGD on 4, 8 or 16 replicas when the rows stay in the 256 MB
//    last-level cache from one call to the next and the thread-per-coordinate
//    kernel has a wavefront for every SIMD (1024 of them): the blocks of the
//    split kernel then run in a few rounds that load and store in step, and
//    that kernel is 3-17 % faster (W = 8, 262,144 coordinates: 7.7 against
//    8.2 us; W = 16: 13.2 against 16.0).  With fewer wavefronts its serial
//    batches cost more (W = 8, 65,539: 4.3 against 3.9), and past the cache
//    the split kernel streams faster (W = 16, 800,001: 52.6 against 46.3);
//  * a DDP step that writes the gradient mean back, past the cache: it streams
//    as many rows in as out and the two are level to 2 % in favour of the
//    thread-per-coordinate kernel (W = 6, 11.2 M: 290 against 296 us); on a
//    small state the split one is twice as fast.
constexpr int64_t kCachedElems = (int64_t)1 << 23;  // W * P: 168 MB of fp32 momentum SGD rows

template <Sync M, Opt O, class PS, class GS, class MS>
constexpr bool kPlainRows = O != Opt::ADAMW && std::is_same<PS, ParamF32>::value &&
                            std::is_same<GS, ParamF32>::value && std::is_same<MS, ParamF32>::value;

template <Sync M, Opt O, class PS, class GS = ParamF32, class MS = ParamF32>
int sync_t(const OptParams& o, const SyncArgs& a) {
    constexpr bool plain = kPlainRows<M, O, PS, GS, MS>;
    const DirectScalars src{o, a.beta, a.alpha * o.lr};
    const bool cached = a.P < kCachedElems / a.W;
    const bool splits = can_split(a.W, blocks_for(a.P), kBlock);
    if constexpr (std::is_same<GS, ParamF32>::value && std::is_same<MS, ParamF32>::value) {
        if (a.flags != 0) {
            const bool split = M != Sync::DDP || !(a.flags & kSyncWriteGbar) || cached;
            return splits && split ? sync_split<M, O, PS, true, GS, MS>(src, a)
                                           : sync_w<M, O, 0, PS, true>(o, a);
        }
    }
    if (a.W == 1) return sync_w<M, O, 1, PS, false, GS, MS>(o, a);
    if (a.W == 2) return sync_w<M, O, 2, PS, false, GS, MS>(o, a);
    if constexpr (plain) {
        if (cached && blocks_for(a.P) >= 1024) {
            if (a.W == 4) return sync_w<M, O, 4, PS, false, GS, MS>(o, a);
            if (a.W == 8) return sync_w<M, O, 8, PS, false, GS, MS>(o, a);
            if (a.W == 16) return sync_w<M, O, 16, PS, false, GS, MS>(o, a);
        }
    }
    if (splits) return sync_split<M, O, PS, false, GS, MS>(src, a);
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
