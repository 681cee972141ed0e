// The synchronisation step with a block's replicas split over its thread
// groups.  Group w (kBlock threads, one wavefront) holds replicas
// w*R .. w*R + R-1 of the block's kCoords coordinates, 4 coordinates a lane,
// and the cross-replica sums go through LDS: every group puts its gradients
// there, sums all W rows itself in the order i = 0, 1, ..., W-1, steps its own
// replicas, puts their new parameters there, and group 0 takes the outer step
// and hands the new model back.  The sums, their order and all arithmetic are
// those of the thread-per-coordinate kernel (sync_chunk), so both give bitwise
// the same state.
//
// Why: a step streams W rows of each family once and is bound by HBM, or, on
// a small state, by how many round trips to memory follow each other.  The
// thread that owns a coordinate of all W replicas runs them in batches, and a
// batch's loads wait for the batch before it (its stores may alias them), so
// it makes W/4 + 2 trips, with the update's divisions of all W replicas in a
// row for AdamW.  Split, all loads of the block are in flight at once, the
// whole step is one trip and three barriers, a thread needs 54-66 registers
// instead of 78-174, and a block's reads are issued together before its
// writes, which the memory takes better.  Measured (us, thread-per-coordinate
// -> split; the 100,003 with a state that is not in the cache):
//   fp32 momentum SGD, W = 8, 23.7 M coordinates      736 -> 706 (5.9 TB/s)
//   fp32 weight decay, W = 16, 23.9 M                1473 -> 1373 (5.9 TB/s)
//   fp32 AdamW, W = 8, 21.3 M                          954 -> 906 (5.7 TB/s)
//   fp32 LocalSGD, W = 12, 2.8 M                       125 -> 114
//   fp32 AdamW, W = 8, 100,003                        16.8 -> 6.9
//   bf16 parameters, W = 32, 2.0 M                     238 -> 189
//   bf16 rows, W = 32, 100,003                          79 -> 14.5
// The 100,003 also gain from the ragged loads, which the kernel on the left did
// not have.  At sizes in between the thread-per-coordinate kernel is the faster
// (cpdp_dispatch.h).
#pragma once

#include "cpdp_device.h"
#include "cpdp_dispatch.h"

namespace cpdp {
namespace {

constexpr int kSplitGroups = kSplitThreads / kBlock;
constexpr int kCoords = kBlock * kVec;  // coordinates of a block

// Orders LDS accesses across the block; global accesses stay in flight (no
// thread uses global memory that another thread of the launch writes).
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ void lds_put(float* row, int lane, const float (&x)[kVec]) {
    *reinterpret_cast<f32x4*>(row + lane * kVec) = f32x4{x[0], x[1], x[2], x[3]};
}

__device__ __forceinline__ void lds_get(const float* row, int lane, float (&x)[kVec]) {
    const f32x4 v = *reinterpret_cast<const f32x4*>(row + lane * kVec);
    x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
}

// s <- the sum over the W rows in LDS, in the order i = 0, 1, ..., W-1, of
// x_i - ref (REF), or of x_i
template <bool REF>
__device__ __forceinline__ void lds_sum(const float* rows, int W, int lane,
                                        const float (&ref)[kVec], float (&s)[kVec]) {
#pragma unroll
    for (int k = 0; k < kVec; ++k) s[k] = 0.0f;
#pragma unroll 4
    for (int i = 0; i < W; ++i) {
        float x[kVec];
        lds_get(rows + i * kCoords, lane, x);
#pragma unroll
        for (int k = 0; k < kVec; ++k) s[k] += REF ? x[k] - ref[k] : x[k];
    }
}

// q0: the block's first coordinate of a row (or plan tensor) of P.  lds: W
// rows of kCoords floats.
template <Sync M, Opt O, int R, class PS, int F, bool EXTRA, class Src, class Rows>
__device__ __forceinline__ void split_chunk(const Src& src, const Rows& r, float* slow,
                                            float* anchor, int W, int64_t q0, int64_t P,
                                            float inv_w, unsigned flags, float* lds) {
    constexpr bool kAdam = O == Opt::ADAMW;
    const int group = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kBlock));
    const int lane = (int)(threadIdx.x % kBlock);
    const bool avg_state = EXTRA && (flags & kSyncAverageState);
    const int64_t p0 = q0 + lane * kVec;
    const int n = F == kFull ? kVec : (int)min(P - p0, (int64_t)kVec);

    // f(c, i) for every replica i = first + c of this group (the last group
    // may hold fewer than R)
    const int first = group * R;
    auto each = [&](auto&& f) {
#pragma unroll
        for (int c = 0; c < R; ++c)
            if (R == 1 || first + c < W) f(c, first + c);
    };

    float g[R][kVec], m[R][kVec], v[R][kVec], th[R][kVec], a[kVec], u[kVec], gbar[kVec], s[kVec];
    each([&](int c, int i) { Rows::GS::template load<F, kNTL>(r.g(i) + p0, n, g[c]); });
    each([&](int c, int i) {
        Rows::MS::template load<F, kNTL>(r.m(i) + p0, n, m[c]);
        if constexpr (kAdam) load_f32<F, kNTL>(r.v(i) + p0, n, v[c]);
        PS::template load<F, kNTL>(r.prm(i) + p0, n, th[c]);
    });
    if constexpr (M == Sync::CPDP) {
        if (group == 0) {
            load_f32<F, kNTL>(anchor + p0, n, a);
            load_f32<F, kNTL>(slow + p0, n, u);
        }
    }
    if constexpr (Src::kDeferred) loads_first();
    StepEntry e;
    if (!src.get(e)) return;  // the same for the whole grid

    // gradient mean (the gradient AllReduce of a synchronisation step)
    if constexpr (M != Sync::LocalSGD) {
        each([&](int c, int i) { lds_put(lds + i * kCoords, lane, g[c]); });
        lds_barrier();
        lds_sum<false>(lds, W, lane, gbar, gbar);
#pragma unroll
        for (int k = 0; k < kVec; ++k) gbar[k] *= inv_w;
        if (EXTRA && (flags & kSyncWriteGbar))
            each([&](int, int i) { Rows::GS::template store<F, kNTS>(r.g(i) + p0, n, gbar); });
        if constexpr (M == Sync::CPDP) lds_barrier();  // the rows are used again below
    }

    // optimizer step of this group's replicas
    each([&](int c, int i) {
#pragma unroll
        for (int k = 0; k < kVec; ++k)
            th[c][k] = opt_update<O, PS, typename Rows::MS>(
                e.o, th[c][k], m[c][k], v[c][k], M == Sync::LocalSGD ? g[c][k] : gbar[k]);
        if constexpr (M != Sync::DDP) lds_put(lds + i * kCoords, lane, th[c]);
    });
    each([&](int c, int i) {
        if (!avg_state) {
            Rows::MS::template store<F, kNTS>(r.m(i) + p0, n, m[c]);
            if constexpr (kAdam) store_f32<F, kNTS>(r.v(i) + p0, n, v[c]);
        }
        if constexpr (M == Sync::DDP) PS::template store<F, kNTS>(r.prm(i) + p0, n, th[c]);
    });

    if constexpr (M != Sync::DDP) {
        lds_barrier();
        if (group == 0) {
            if constexpr (M == Sync::CPDP) {
                lds_sum<true>(lds, W, lane, a, s);
                slowmo_step(e.beta, e.alpha_lr, e.o.lr, inv_w, s, u, a);
                store_f32<F, kNTS>(slow + p0, n, u);
                store_f32<F, kNTS>(anchor + p0, n, a);
            } else {
                float x0[kVec];
                lds_get(lds, lane, x0);
                lds_sum<true>(lds, W, lane, x0, s);
#pragma unroll
                for (int k = 0; k < kVec; ++k) a[k] = fmaf(s[k], inv_w, x0[k]);
                if (anchor != nullptr) store_f32<F, kNTS>(anchor + p0, n, a);
            }
            lds_put(lds, lane, a);  // only this group's own lanes read row 0 before
        }
        lds_barrier();
        lds_get(lds, lane, a);
        each([&](int, int i) { PS::template store<F, kNTS>(r.prm(i) + p0, n, a); });
    }

    if constexpr (EXTRA) {
        if (avg_state) {
            // every group takes the mean of the replicas' state for itself
            auto mean = [&](float (&x)[R][kVec]) {
                lds_barrier();  // earlier reads of the rows are done
                each([&](int c, int i) { lds_put(lds + i * kCoords, lane, x[c]); });
                lds_barrier();
                lds_sum<false>(lds, W, lane, s, s);
#pragma unroll
                for (int k = 0; k < kVec; ++k) s[k] *= inv_w;
            };
            mean(m);
            each([&](int, int i) { Rows::MS::template store<F, kNTS>(r.m(i) + p0, n, s); });
            if constexpr (kAdam) {
                mean(v);
                each([&](int, int i) { store_f32<F, kNTS>(r.v(i) + p0, n, s); });
            }
        }
    }
}

// split_chunk with the way the block's lanes move their coordinates
template <Sync M, Opt O, int R, class PS, bool EXTRA, class Src, class Rows>
__device__ __forceinline__ void split_dispatch(const Src& src, const Rows& r, float* slow,
                                               float* anchor, int W, int64_t q0, int64_t P,
                                               float inv_w, unsigned flags, float* lds) {
    if (q0 + kCoords <= P)
        split_chunk<M, O, R, PS, kFull, EXTRA>(src, r, slow, anchor, W, q0, P, inv_w, flags, lds);
    else if (P >= kVec)
        split_chunk<M, O, R, PS, kRagged, EXTRA>(src, r, slow, anchor, W, q0, P, inv_w, flags,
                                                 lds);
    else
        split_chunk<M, O, R, PS, kTiny, EXTRA>(src, r, slow, anchor, W, q0, P, inv_w, flags, lds);
}

// The step as the dispatch rules see it.
template <Sync M, Opt O, class PS, class GS = ParamF32, class MS = ParamF32>
constexpr StepKind step_kind() {
    return {M, O, std::is_same<PS, ParamBF16>::value, std::is_same<MS, ParamBF16>::value,
            std::is_same<GS, ParamBF16>::value};
}

// Replicas a group holds: one up to 16 groups, then two, or four where the
// parameters are bf16 and a row is half as long (all-bf16 DDP, 32 x 262,140: 24 us
// with four, 27 with two).  AdamW takes two all the same (24 x 2.7 M, bf16
// parameters: 324 us with two, 349 with four).
template <Opt O, class PS, class Launch>
int with_split_r(int W, Launch launch_r) {
    if (W <= kSplitGroups) return launch_r(std::integral_constant<int, 1>());
    constexpr bool kFour = std::is_same<PS, ParamBF16>::value && O != Opt::ADAMW;
    return launch_r(std::integral_constant<int, kFour ? 4 : 2>());
}

template <class... Args>
int launch_split(void (*kernel)(Args...), int64_t blocks, int W, int R, void* stream,
                 typename same_type<Args>::type... args) {
    void* argv[] = {static_cast<void*>(&args)...};
    return (int)hipLaunchKernel(reinterpret_cast<const void*>(kernel), dim3((unsigned)blocks),
                                dim3((unsigned)split_threads(W, R, kBlock)), argv,
                                (size_t)W * kCoords * sizeof(float),
                                static_cast<hipStream_t>(stream));
}

// Wavefronts a SIMD has to hold.  With two replicas a group the block is up to 16
// wavefronts; AdamW took 66 registers then, which leaves room for one such block
// a CU where 64 leave room for two (32 x 513,800 coordinates: 107 us, so 87).
constexpr int split_waves(int R) { return R == 2 ? 8 : 1; }

// ---- flat layout -------------------------------------------------------------------

template <Sync M, Opt O, int R, class PS, bool EXTRA, class GS, class MS, class Src>
__global__ __launch_bounds__(kSplitThreads, split_waves(R)) void sync_split_kernel(
    Src src, typename PS::T* __restrict__ params, typename MS::T* __restrict__ mom,
    float* __restrict__ mom2, GradPtr<EXTRA, GS> __restrict__ grads, float* __restrict__ slow,
    float* __restrict__ anchor, int W, int64_t ld, int64_t P, float inv_w, unsigned flags) {
    extern __shared__ __align__(16) float lds[];
    // Strided holds mutable row pointers; without EXTRA no store to the
    // gradient rows is instantiated
    const Strided<PS, GS, MS> r{params, mom, mom2, const_cast<typename GS::T*>(grads), ld};
    split_dispatch<M, O, R, PS, EXTRA>(src, r, slow, anchor, W, (int64_t)blockIdx.x * kCoords, P,
                                       inv_w, flags, lds);
}

template <Sync M, Opt O, class PS, bool EXTRA, class GS, class MS, class Src>
int sync_split(const Src& src, const SyncArgs& a) {
    using T = typename PS::T;
    // the variants run only from the entry points whose gradient argument is
    // mutable (flags != 0), so dropping const here restores the caller's type
    const GradPtr<EXTRA, GS> grads =
        const_cast<typename GS::T*>(static_cast<const typename GS::T*>(a.grads));
    return with_split_r<O, PS>(a.W, [&](auto R) {
        return launch_split(sync_split_kernel<M, O, R, PS, EXTRA, GS, MS, Src>, blocks_for(a.P),
                            a.W, R, a.stream, src, static_cast<T*>(a.params),
                            static_cast<typename MS::T*>(a.mom), a.mom2, grads, a.slow, a.anchor,
                            a.W, a.ld, a.P, 1.0f / (float)a.W, a.flags);
    });
}

}  // namespace
}  // namespace cpdp
