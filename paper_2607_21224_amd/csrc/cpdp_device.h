// Device building blocks of the gfx950 kernels of the CPDP reconcile hot path
// (state initialisation, the local optimizer step, and the fused
// synchronisation step of the three strategies -- CPDP reconcile, LocalSGD
// averaging, DDP gradient step -- each for momentum SGD, SGD with weight
// decay, or AdamW).  The kernels and their launchers live in the kernels_*.hip
// translation units, which are compiled in parallel; everything here is
// templates and inline functions in an anonymous namespace, so each unit
// instantiates only what it launches.
//
// All of them are HBM-streaming kernels: nothing here is a dense contraction, so
// there is no MFMA.  Every thread owns VEC = 4 consecutive coordinates and moves
// them with 128-bit (fp32) or 64-bit (bf16) vector accesses (parameters, and on
// the plain momentum-SGD entry points also the gradients and the momentum, may
// be stored as bf16); a wavefront therefore touches 1 KiB (fp32) of each array
// row per access, fully coalesced.  Every output element is written by exactly
// one thread, there are no atomics and no inter-block dependencies, and the
// cross-replica sums run in a fixed order (replica 0, 1, ..., W-1), whether one
// thread holds a coordinate of all replicas (sync_chunk) or a block's wavefronts
// hold one each and meet in LDS (split_chunk), so results are bitwise
// independent of the launch shape.
//
// Arithmetic is fp32 with explicit fmaf in the optimizer updates and the
// SlowMo step (the library is built with -ffp-contract=off so nothing else is
// fused).  bf16 parameters are widened on load and rounded to nearest-even on
// every store, including the x_i fed to the parameter mean, where the
// framework implementation writes the optimizer's result to the parameter
// tensor before averaging it (Sec. 4.2).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "cpdp_launch.h"

namespace cpdp {
namespace {

// One wavefront per block (the split step: per thread group).  On MI355X
// 64-thread blocks ran the thread-per-coordinate reconcile 2.6-3.1 % and the
// local step 1-3.7 % faster than 256-thread blocks on the fp32 ResNet-50 /
// ViT-S sized states (level on the 32-replica bf16 state); a kernel streaming
// the reconcile's rows with no arithmetic gains as much, so the difference is
// in how the memory system sees the blocks, not in the code.  Results do not depend
// on it (every thread owns its 4 coordinates).
#ifndef CPDP_BLOCK
#define CPDP_BLOCK 64
#endif
constexpr int kBlock = CPDP_BLOCK;
constexpr int kVec = 4;

// State tensors are streamed exactly once per call; nontemporal accesses keep
// them from displacing anything useful in L2 / MALL.
#ifndef CPDP_NT_LOAD
#define CPDP_NT_LOAD 1
#endif
#ifndef CPDP_NT_STORE
#define CPDP_NT_STORE 1
#endif
constexpr bool kNTL = CPDP_NT_LOAD != 0;
constexpr bool kNTS = CPDP_NT_STORE != 0;

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

template <bool NT, class V>
__device__ __forceinline__ V vload(const V* p) {
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}

template <bool NT, class V>
__device__ __forceinline__ void vstore(V* p, V v) {
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}

// ---- a lane's 4 coordinates ------------------------------------------------
//
// A lane covers up to 4 coordinates of a row of P, of which n = min(4, P - p)
// exist (n may be zero or negative for lanes of a ragged block past the row's
// end).  Three ways to move them:
//   kFull    n = 4 for every lane of the wavefront: 128-bit (bf16: 64-bit)
//            accesses.
//   kRagged  P >= 4, the row's last wavefront: every lane loads 4 existing
//            coordinates with one access, the ones past the end taking the
//            row's last 4 (aligned to the element only) and shifting theirs
//            into place.  The last 4 may belong to another lane, wavefront or
//            block that has already updated them; what was loaded of them is
//            dropped.  Loading the short lane's coordinates one by one behind
//            a branch made a wave wait for each before it issued the next, W
//            round trips to memory in a row (reconcile of 8 x 100,003 bf16
//            coordinates: 15.0 us, so 8.9, both with the thread-per-coordinate
//            kernel).
//   kTiny    P < 4: one by one, the missing ones taking the last coordinate.
//            Every kernel carries this code, so it must not cost the others
//            registers: with the loads of a batch of replicas in flight, each
//            with an address of its own, the run-time-W kernel needed 138
//            registers for momentum SGD and 202 for AdamW (3 and 2 wavefronts a
//            SIMD) instead of 78 and 117 (6 and 4).  So the loads are issued in
//            order, and sync_chunk takes one replica at a time.
// Nothing computed from a missing coordinate is stored.
enum Lanes { kTiny, kFull, kRagged };

typedef float f32x4_el __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x2_el __attribute__((ext_vector_type(2), aligned(2)));

__device__ __forceinline__ int tail_index(int k, int n) { return k < n ? k : n - 1; }

// x[k] <- x[k + shift] (the last one past the end)
__device__ __forceinline__ void shift_down(int shift, float (&x)[kVec]) {
    const float a = x[0], b = x[1], c = x[2], d = x[3];
    x[0] = shift == 0 ? a : shift == 1 ? b : shift == 2 ? c : d;
    x[1] = shift == 0 ? b : shift == 1 ? c : d;
    x[2] = shift == 0 ? c : d;
}

template <int F, bool NT>
__device__ __forceinline__ void load_f32(const float* p, int n, float (&x)[kVec]) {
    if constexpr (F == kFull) {
        f32x4 v = vload<NT>(reinterpret_cast<const f32x4*>(p));
        x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
    } else if constexpr (F == kRagged) {
        const f32x4_el v = *reinterpret_cast<const f32x4_el*>(p - (kVec - n));
        x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
        shift_down(kVec - n, x);
    } else {
#pragma unroll
        for (int k = 0; k < kVec; ++k) {
            x[k] = p[tail_index(k, n)];
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

template <int F, bool NT>
__device__ __forceinline__ void store_f32(float* p, int n, const float (&x)[kVec]) {
    if (F == kFull || (F == kRagged && n == kVec)) {
        f32x4 v = {x[0], x[1], x[2], x[3]};
        vstore<NT>(reinterpret_cast<f32x4*>(p), v);
    } else {
#pragma unroll
        for (int k = 0; k < kVec; ++k)
            if (k < n) p[k] = x[k];
    }
}

// body(lanes, n) with the way the calling wavefront's lanes move their
// coordinates p0 .. p0 + n - 1 of a row of P (p0 is its lane's first)
template <class Body>
__device__ __forceinline__ void for_lanes(int64_t p0, int64_t P, Body body) {
    if (__all(p0 + kVec <= P))
        body(std::integral_constant<int, kFull>(), kVec);
    else if (P >= kVec)
        body(std::integral_constant<int, kRagged>(), (int)min(P - p0, (int64_t)kVec));
    else
        body(std::integral_constant<int, kTiny>(), (int)min(P - p0, (int64_t)kVec));
}

// ---- parameter storage ----------------------------------------------------

struct ParamF32 {
    using T = float;
    __device__ static __forceinline__ float round(float x) { return x; }
    template <int F, bool NT>
    __device__ static __forceinline__ void load(const T* p, int n, float (&x)[kVec]) {
        load_f32<F, NT>(p, n, x);
    }
    template <int F, bool NT>
    __device__ static __forceinline__ void store(T* p, int n, const float (&x)[kVec]) {
        store_f32<F, NT>(p, n, x);
    }
};

// Both results are computed and one is selected: with an early return for NaN
// the compiler puts a branch around the values it rounds where the code is large
// (reconcile of 4 x 16,380 coordinates, bf16 parameters, thread-per-coordinate
// kernel: 3.3 us with the branches, 2.6 without; of 32 x 1,000,000 all-bf16 ones,
// split: 90 and 84).
__device__ __forceinline__ uint32_t bf16_bits(float f) {
    const uint32_t b = __float_as_uint(f);
    const uint32_t quiet = (b >> 16) | 0x40u;                         // a quiet NaN
    const uint32_t nearest = (b + 0x7FFFu + ((b >> 16) & 1u)) >> 16;  // ties even
    return (b & 0x7FFFFFFFu) > 0x7F800000u ? quiet : nearest;
}

__device__ __forceinline__ float bf16_value(uint32_t h) { return __uint_as_float(h << 16); }

struct ParamBF16 {
    using T = uint16_t;
    __device__ static __forceinline__ float round(float x) { return bf16_value(bf16_bits(x)); }
    template <int F, bool NT>
    __device__ static __forceinline__ void load(const T* p, int n, float (&x)[kVec]) {
        if constexpr (F != kTiny) {
            u32x2 v;
            if constexpr (F == kFull)
                v = vload<NT>(reinterpret_cast<const u32x2*>(p));
            else
                v = *reinterpret_cast<const u32x2_el*>(p - (kVec - n));
            x[0] = __uint_as_float(v.x << 16);
            x[1] = __uint_as_float(v.x & 0xFFFF0000u);
            x[2] = __uint_as_float(v.y << 16);
            x[3] = __uint_as_float(v.y & 0xFFFF0000u);
            if constexpr (F == kRagged) shift_down(kVec - n, x);
        } else {
#pragma unroll
            for (int k = 0; k < kVec; ++k) {
                x[k] = bf16_value(p[tail_index(k, n)]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    template <int F, bool NT>
    __device__ static __forceinline__ void store(T* p, int n, const float (&x)[kVec]) {
        if (F == kFull || (F == kRagged && n == kVec)) {
            u32x2 v = {bf16_bits(x[0]) | (bf16_bits(x[1]) << 16),
                       bf16_bits(x[2]) | (bf16_bits(x[3]) << 16)};
            vstore<NT>(reinterpret_cast<u32x2*>(p), v);
        } else {
#pragma unroll
            for (int k = 0; k < kVec; ++k)
                if (k < n) p[k] = (uint16_t)bf16_bits(x[k]);
        }
    }
};

// ---- the per-replica optimizer update -------------------------------------------
//
// One coordinate of one replica: th is the stored parameter (widened), m / v
// the optimizer state, g the gradient the update uses.  Returns the new
// parameter, rounded to the parameter storage type (the value the optimizer
// writes to the parameter tensor).
//   SGD     m <- mu m + g;              th <- th - lr m
//   SGD_WD  d = g + wd th;  m <- mu m + d;  th <- th - lr m      (coupled L2)
//   ADAMW   th <- round(th (1 - lr wd));  m <- b1 m + (1-b1) g;
//           v <- b2 v + (1-b2) g^2;
//           th <- th - (lr / (1-b1^t)) m / (sqrt(v) / sqrt(1-b2^t) + eps)
// The AdamW bias-correction factors and the decay factor are folded into
// OptParams on the host (they depend on the step count only) and enter the
// arithmetic as fp32 values, as they do in the framework's fp32 tensor ops.

template <Opt O, class PS, class MS = ParamF32>
__device__ __forceinline__ float opt_update(const OptParams& o, float th, float& m, float& v,
                                            float g) {
    // the momentum buffer is stored (rounded to its storage type MS) before
    // the parameter update reads it, as the framework's in-place buffer does
    if constexpr (O == Opt::SGD) {
        m = MS::round(fmaf(o.mu, m, g));
        return PS::round(fmaf(-o.lr, m, th));
    } else if constexpr (O == Opt::SGD_WD) {
        const float d = fmaf(o.wd, th, g);
        m = MS::round(fmaf(o.mu, m, d));
        return PS::round(fmaf(-o.lr, m, th));
    } else {
        const float t = PS::round(th * o.decay);
        m = fmaf(o.omb1, g, o.mu * m);
        v = fmaf(o.omb2, g * g, o.beta2 * v);
        const float denom = sqrtf(v) / o.sqrt_bc2 + o.eps;
        return PS::round(fmaf(-o.step_size, m / denom, t));
    }
}

// SlowMo outer step of 4 coordinates, s the sum of x_i - a:
//   u <- beta u + (a - avg)/lr ;  a <- a - alpha lr u
__device__ __forceinline__ void slowmo_step(float beta, float alpha_lr, float lr, float inv_w,
                                            const float (&s)[kVec], float (&u)[kVec],
                                            float (&a)[kVec]) {
#pragma unroll
    for (int k = 0; k < kVec; ++k) {
        const float drift = s[k] * inv_w;  // avg - a
        u[k] = fmaf(beta, u[k], -drift / lr);
        a[k] = fmaf(-alpha_lr, u[k], a[k]);
    }
}

// ---- replica addressing ------------------------------------------------------------
//
// Where replica i's row of each family starts.  Strided is the flat layout of
// the C ABI (base + i*ld); Table is a multi-tensor plan (one device pointer
// per replica and tensor, replica-major).  Both expose the same accessors, so
// the step code below is written once.

template <class PS, class GS_ = ParamF32, class MS_ = ParamF32>
struct Strided {
    using GS = GS_;  // gradient storage type
    using MS = MS_;  // momentum storage type
    typename PS::T* params;
    typename MS::T* mom;
    float* mom2;
    typename GS::T* grads;
    int64_t ld;
    __device__ __forceinline__ typename PS::T* prm(int i) const { return params + (int64_t)i * ld; }
    __device__ __forceinline__ typename MS::T* m(int i) const { return mom + (int64_t)i * ld; }
    __device__ __forceinline__ float* v(int i) const { return mom2 + (int64_t)i * ld; }
    __device__ __forceinline__ typename GS::T* g(int i) const { return grads + (int64_t)i * ld; }
};

// An address from a plan table as a pointer to global memory.  A plain cast of
// the integer makes a generic pointer, whose flat accesses also wait on the LDS
// counter.
template <class T>
__device__ __forceinline__ T* global_ptr(int64_t addr) {
    return (T*)(T __attribute__((address_space(1)))*)addr;
}

template <class PS>
struct Table {
    using GS = ParamF32;    // plans hold fp32 gradients
    using MS = ParamF32;    // and fp32 momentum
    const int64_t* params;  // 64-bit device addresses, entry i*n + t
    const int64_t* mom;
    const int64_t* mom2;
    const int64_t* grads;
    int64_t n, t;
    __device__ __forceinline__ typename PS::T* prm(int i) const {
        return global_ptr<typename PS::T>(params[i * n + t]);
    }
    __device__ __forceinline__ float* m(int i) const { return global_ptr<float>(mom[i * n + t]); }
    __device__ __forceinline__ float* v(int i) const { return global_ptr<float>(mom2[i * n + t]); }
    __device__ __forceinline__ float* g(int i) const { return global_ptr<float>(grads[i * n + t]); }
};

// The sections of a plan table (layout documented in cpdp_launch.h).
struct PlanView {
    const int64_t* chunk_start;
    const int64_t* numel;
    const int64_t* params;
    const int64_t* mom;
    const int64_t* mom2;
    const int64_t* grads;
    const int64_t* slow;
    const int64_t* anchor;
};

__device__ __forceinline__ PlanView plan_view(const int64_t* plan, int64_t W, int64_t n) {
    PlanView v;
    v.chunk_start = plan + kPlanHeaderWords;
    v.numel = v.chunk_start + (n + 1);
    v.params = v.numel + n;
    v.mom = v.params + W * n;
    v.mom2 = v.mom + W * n;
    v.grads = v.mom2 + W * n;
    v.slow = v.grads + W * n;
    v.anchor = v.slow + n;
    return v;
}

// tensor holding chunk b: the largest t < n with chunk_start[t] <= b (an
// empty tensor never qualifies as the last such t, since b < chunk_start[n]).
// Called by whole wavefronts: the 64 lanes look at 64 evenly spaced starts at
// once, so 161 tensors take two dependent loads where a binary search by every
// thread took eight, each a trip to L2 or beyond before the first data load
// could be issued (AdamW reconcile of 4 x 271,117 coordinates in 62
// tensors, not in the cache, with the split step: 13.5 -> 9.1 us).
__device__ __forceinline__ int64_t plan_tensor(const PlanView& v, int n, int64_t b) {
    const int lane = (int)(threadIdx.x % 64);
    int lo = 0, hi = n;  // chunk_start[lo] <= b < chunk_start[hi]
    while (hi - lo > 1) {
        const int step = (hi - lo + 63) / 64;
        const int at = lo + lane * step;
        const bool le = at < hi && v.chunk_start[at] <= b;
        lo += (__popcll(__ballot(le)) - 1) * step;  // starts do not decrease: a prefix of lanes
        hi = min(hi, lo + step);
    }
    return lo;
}

// The same by a binary search with scalar loads: a longer chain, but one that
// costs the vector memory path nothing.
__device__ __forceinline__ int64_t plan_tensor_scalar(const PlanView& v, int n, int64_t b) {
    int lo = 0, hi = n;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (v.chunk_start[mid] <= b) lo = mid;
        else hi = mid;
    }
    return lo;
}

// ---- block order of the local step ---------------------------------------------
//
// The local step's blocks are the cells (replica row, column of kBlock * kVec
// coordinates) of a W x columns grid, taken in plain replica-major order: the
// hardware hands workgroup b of a launch to XCD b % 8, so each XCD streams
// every eighth column.  Dealing the blocks to the XCDs in contiguous eighths
// of the state instead was 4-5 % faster for the momentum-SGD update with
// 256-thread blocks, but 0.6-2.9 % slower with the 64-thread blocks used
// here (and level for AdamW), so the plain order stays.

// blocks of a local-step launch over `cells` cells
inline int64_t local_grid(int64_t cells) { return cells; }

// the cell of this block, or -1 for a block past the last cell
__device__ __forceinline__ int64_t local_cell(int64_t cells) {
    return (int64_t)blockIdx.x < cells ? (int64_t)blockIdx.x : -1;
}

// ---- step tables: the scalars of the current step read from device memory -----
//
// Every thread reads the position word and the entry `ahead` places past it (the
// same addresses for the whole grid, so they are served from cache).  A position
// outside the table means the table is used up: the kernel returns without
// touching the state, so replaying a captured graph past its table cannot run a
// step with undefined scalars.

// The table does not change while a step runs, so it is read through the
// constant address space (scalar loads, which do not wait for the data).
__device__ __forceinline__ bool step_entry(const int64_t* table, int64_t ahead,
                                           StepEntry& e) {
    typedef const int64_t __attribute__((address_space(4))) Word;
    typedef const StepEntry __attribute__((address_space(4))) Entry;
    Word* t = (Word*)table;
    const int64_t pos = t[0] + ahead, n = t[1];
    if ((uint64_t)pos >= (uint64_t)n) return false;
    Entry* at = (Entry*)(t + kStepTableHeaderWords) + pos;
    e.o = {at->o.lr, at->o.mu, at->o.wd, at->o.omb1, at->o.beta2,
           at->o.omb2, at->o.eps, at->o.step_size, at->o.sqrt_bc2, at->o.decay};
    e.beta = at->beta;
    e.alpha_lr = at->alpha_lr;
    return true;
}

// Keeps the loads written before it ahead of what follows: the compiler would
// move them past the test of a table's position, behind its two dependent loads.
__device__ __forceinline__ void loads_first() { asm volatile("" ::: "memory"); }

// Where a step's scalars come from: the launch arguments, or the entry at the
// position of a device step table (no entry when the table is used up).
struct DirectScalars {
    static constexpr bool kDeferred = false;
    OptParams o;
    float beta;
    float alpha_lr;
    __device__ __forceinline__ bool get(StepEntry& e) const {
        e.o = o;
        e.beta = beta;
        e.alpha_lr = alpha_lr;
        return true;
    }
};

struct TableScalars {
    static constexpr bool kDeferred = true;
    const int64_t* table;
    int64_t ahead;  // entries past the position
    __device__ __forceinline__ bool get(StepEntry& e) const { return step_entry(table, ahead, e); }
};

// ---- local step: one replica row per block, 4 coordinates per thread -------

template <Opt O, class PS, class GS, class MS, int F, class Src>
__device__ __forceinline__ void local_chunk(const Src& src, typename PS::T* params,
                                            typename MS::T* mom, float* mom2,
                                            const typename GS::T* grads, int n) {
    float g[kVec], m[kVec], v[kVec] = {0.0f, 0.0f, 0.0f, 0.0f}, th[kVec];
    GS::template load<F, kNTL>(grads, n, g);
    MS::template load<F, kNTL>(mom, n, m);
    if constexpr (O == Opt::ADAMW) load_f32<F, kNTL>(mom2, n, v);
    PS::template load<F, kNTL>(params, n, th);
    // a table's entry is two dependent loads away: look while the data comes
    if constexpr (Src::kDeferred) loads_first();
    StepEntry e;
    if (!src.get(e)) return;
#pragma unroll
    for (int k = 0; k < kVec; ++k) th[k] = opt_update<O, PS, MS>(e.o, th[k], m[k], v[k], g[k]);
    MS::template store<F, kNTS>(mom, n, m);
    if constexpr (O == Opt::ADAMW) store_f32<F, kNTS>(mom2, n, v);
    PS::template store<F, kNTS>(params, n, th);
}

template <Opt O, class PS, class GS = ParamF32, class MS = ParamF32, class Src>
__device__ __forceinline__ void local_dispatch(const Src& src, typename PS::T* params,
                                               typename MS::T* mom, float* mom2,
                                               const typename GS::T* grads, int64_t p0,
                                               int64_t P) {
    for_lanes(p0, P, [&](auto lanes, int n) {
        local_chunk<O, PS, GS, MS, lanes>(src, params + p0, mom + p0, mom2 + p0, grads + p0, n);
    });
}

// ---- fused synchronisation steps ----------------------------------------------
//
// One thread owns 4 coordinates across all W replicas.  WT > 0 fixes W at
// compile time (fully unrolled); otherwise W is taken at run time (batches of
// kChunk, then single replicas).  Within a batch all loads are issued before
// any store.  The batching matters because the compiler cannot prove that two
// replica rows never alias (ld is a run-time value, plan pointers are data),
// so a store for replica i would otherwise hold back the loads of replica
// i+1 and the thread would wait one round trip to HBM per replica.
//
// Sync::CPDP      gradient mean, synchronized optimizer step, parameter mean,
//                 SlowMo, copy-back (the reconcile).
// Sync::LocalSGD  each replica steps on its own gradient, then the parameter
//                 mean is copied back (no gradient mean, no SlowMo).
// Sync::DDP       gradient mean and the same optimizer step on every replica,
//                 no parameter mean.
//
// EXTRA = true enables the optional variants selected by `flags` (run-time W
// only): kSyncWriteGbar stores the gradient mean into every gradient row;
// kSyncAverageState replaces every replica's optimizer state by the replica
// mean after the step.

// Replica batch of the synchronisation steps.  With 64-thread blocks,
// batches of 4 were level with or up to 1.5 % faster than batches of 8 (and
// batches of 2 slower) on the reconcile of the four full-size states; the
// batching does not change the arithmetic or its order.
#ifndef CPDP_RECON_CHUNK
#define CPDP_RECON_CHUNK 4
#endif
constexpr int kChunk = CPDP_RECON_CHUNK;

// per-thread values carried across replica batches
struct SyncAcc {
    float gbar[kVec];  // gradient mean
    float a[kVec];     // anchor (CPDP) / averaged model (LocalSGD)
    float u[kVec];     // SlowMo state
    float s[kVec];     // sum of x_i - reference
    float x0[kVec];    // LocalSGD reference: replica 0's x
    float msum[kVec];  // optimizer-state sums (state reconciliation)
    float vsum[kVec];
};

template <int C, int F, class Rows>
__device__ __forceinline__ void grad_batch(const Rows& r, int i0, int64_t p0, int n,
                                           float (&acc)[kVec]) {
    float g[C][kVec];
#pragma unroll
    for (int c = 0; c < C; ++c)
        Rows::GS::template load<F, kNTL>(r.g(i0 + c) + p0, n, g[c]);
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
        for (int k = 0; k < kVec; ++k) acc[k] += g[c][k];
}

template <Sync M, Opt O, int C, class PS, int F, class Rows>
__device__ __forceinline__ void step_batch(const OptParams& o, const Rows& r, int i0, int64_t p0,
                                           int n, SyncAcc& z, bool avg_state) {
    constexpr bool kAdam = O == Opt::ADAMW;
    float m[C][kVec], v[C][kVec], th[C][kVec], g[C][kVec];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        if constexpr (M == Sync::LocalSGD)
            Rows::GS::template load<F, kNTL>(r.g(i0 + c) + p0, n, g[c]);
        Rows::MS::template load<F, kNTL>(r.m(i0 + c) + p0, n, m[c]);
        if constexpr (kAdam) load_f32<F, kNTL>(r.v(i0 + c) + p0, n, v[c]);
        PS::template load<F, kNTL>(r.prm(i0 + c) + p0, n, th[c]);
    }
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
        for (int k = 0; k < kVec; ++k) {
            const float gk = M == Sync::LocalSGD ? g[c][k] : z.gbar[k];
            const float x = opt_update<O, PS, typename Rows::MS>(o, th[c][k], m[c][k], v[c][k],
                                                                 gk);
            if constexpr (M == Sync::CPDP) {
                z.s[k] += x - z.a[k];
            } else if constexpr (M == Sync::LocalSGD) {
                if (i0 + c == 0) z.x0[k] = x;
                z.s[k] += x - z.x0[k];
            } else {
                th[c][k] = x;
            }
        }
#pragma unroll
    for (int c = 0; c < C; ++c) {
        if (avg_state) {
#pragma unroll
            for (int k = 0; k < kVec; ++k) {
                z.msum[k] += m[c][k];
                if constexpr (kAdam) z.vsum[k] += v[c][k];
            }
        } else {
            Rows::MS::template store<F, kNTS>(r.m(i0 + c) + p0, n, m[c]);
            if constexpr (kAdam) store_f32<F, kNTS>(r.v(i0 + c) + p0, n, v[c]);
        }
        if constexpr (M == Sync::DDP) PS::template store<F, kNTS>(r.prm(i0 + c) + p0, n, th[c]);
    }
}

template <Sync M, Opt O, int WT, class PS, int F, bool EXTRA, class Rows>
__device__ __forceinline__ void sync_chunk(const OptParams& o, const Rows& r, float* slow,
                                           float* anchor, int W, int64_t p0, int n, float beta,
                                           float alpha_lr, float inv_w, unsigned flags) {
    static_assert(!EXTRA || WT <= 0, "variants run on the run-time-W kernel");
    // rows of fewer than 4 coordinates take their replicas one at a time
    constexpr bool kUnroll = WT > 0 && F != kTiny;
    constexpr int C = F == kTiny ? 1 : WT > 0 ? (WT < kChunk ? WT : kChunk) : kChunk;
    static_assert(WT <= 0 || WT % C == 0, "replica batches must tile W");
    constexpr bool kAdam = O == Opt::ADAMW;
    const int nw = WT > 0 ? WT : W;
    const bool avg_state = EXTRA && (flags & kSyncAverageState);
    SyncAcc z;
#pragma unroll
    for (int k = 0; k < kVec; ++k)
        z.gbar[k] = z.a[k] = z.u[k] = z.s[k] = z.x0[k] = z.msum[k] = z.vsum[k] = 0.0f;

    // gradient mean (the gradient AllReduce of a synchronisation step),
    // summed in the fixed order i = 0, 1, ..., W-1
    if constexpr (M != Sync::LocalSGD) {
        float acc[kVec] = {0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (kUnroll) {
#pragma unroll
            for (int i0 = 0; i0 < WT; i0 += C) grad_batch<C, F>(r, i0, p0, n, acc);
        } else {
            int i0 = 0;
            if constexpr (C > 1)
                for (; i0 + C <= nw; i0 += C) grad_batch<C, F>(r, i0, p0, n, acc);
#pragma nounroll
            for (; i0 < nw; ++i0) grad_batch<1, F>(r, i0, p0, n, acc);
        }
#pragma unroll
        for (int k = 0; k < kVec; ++k) z.gbar[k] = acc[k] * inv_w;
        if (EXTRA && (flags & kSyncWriteGbar))
            for (int i = 0; i < nw; ++i)
                Rows::GS::template store<F, kNTS>(r.g(i) + p0, n, z.gbar);
    }

    if constexpr (M == Sync::CPDP) {
        load_f32<F, kNTL>(anchor + p0, n, z.a);
        load_f32<F, kNTL>(slow + p0, n, z.u);
    }

    // optimizer step of every replica.  The parameter mean is accumulated as
    // a sum of differences to a reference that is close to every x_i (the
    // anchor for CPDP, replica 0's x for LocalSGD), so the small deviations
    // keep their precision.
    if constexpr (kUnroll) {
#pragma unroll
        for (int i0 = 0; i0 < WT; i0 += C)
            step_batch<M, O, C, PS, F>(o, r, i0, p0, n, z, avg_state);
    } else {
        int i0 = 0;
        if constexpr (C > 1)
            for (; i0 + C <= nw; i0 += C) step_batch<M, O, C, PS, F>(o, r, i0, p0, n, z, avg_state);
#pragma nounroll
        for (; i0 < nw; ++i0) step_batch<M, O, 1, PS, F>(o, r, i0, p0, n, z, avg_state);
    }
    if (avg_state) {
#pragma unroll
        for (int k = 0; k < kVec; ++k) {
            z.msum[k] *= inv_w;
            z.vsum[k] *= inv_w;
        }
        for (int i = 0; i < nw; ++i) {
            Rows::MS::template store<F, kNTS>(r.m(i) + p0, n, z.msum);
            if constexpr (kAdam) store_f32<F, kNTS>(r.v(i) + p0, n, z.vsum);
        }
    }
    if constexpr (M == Sync::DDP) return;

    if constexpr (M == Sync::CPDP) {
        slowmo_step(beta, alpha_lr, o.lr, inv_w, z.s, z.u, z.a);
        store_f32<F, kNTS>(slow + p0, n, z.u);
        store_f32<F, kNTS>(anchor + p0, n, z.a);
    } else {
#pragma unroll
        for (int k = 0; k < kVec; ++k) z.a[k] = fmaf(z.s[k], inv_w, z.x0[k]);
        if (anchor != nullptr) store_f32<F, kNTS>(anchor + p0, n, z.a);
    }

    // copy the reconciled model back into every replica
#pragma unroll
    for (int i = 0; i < nw; ++i) PS::template store<F, kNTS>(r.prm(i) + p0, n, z.a);
}

// The gradient rows are written only by the variants (the gradient-mean
// write-back), so only those instantiations take them as mutable.
template <bool EXTRA, class GS = ParamF32>
using GradPtr = typename std::conditional<EXTRA, typename GS::T*, const typename GS::T*>::type;

// ---- launch helpers -------------------------------------------------------------

inline int64_t blocks_for(int64_t P) {
    return (P + (int64_t)kBlock * kVec - 1) / ((int64_t)kBlock * kVec);
}

template <class T>
struct same_type {
    using type = T;
};

// LDS that a block of kBlock threads reserves so that at most `waves` wavefronts a
// SIMD are resident (0: as many as fit): a CU has 160 KB, handed out in units of
// 1280 bytes, and a block may ask for 64 KB.
constexpr size_t lds_for_waves(int waves) {
    if (waves == 0) return 0;
    const size_t share = (size_t)160 * 1024 * (kBlock / 64) / (4 * waves) / 1280 * 1280;
    return share < 65536 ? share : 65536;
}

// Argument types come from the kernel's signature only (the trailing
// parameters are a non-deduced context), so every argument is converted to
// exactly what the kernel takes before its address goes into argv.
template <class... Args>
int launch_resident(int waves, void (*kernel)(Args...), int64_t blocks, void* stream,
                    typename same_type<Args>::type... args) {
    void* argv[] = {static_cast<void*>(&args)...};
    hipError_t e = hipLaunchKernel(reinterpret_cast<const void*>(kernel),
                                   dim3((unsigned)blocks), dim3(kBlock), argv,
                                   lds_for_waves(waves), static_cast<hipStream_t>(stream));
    return (int)e;
}

template <class... Args>
int launch(void (*kernel)(Args...), int64_t blocks, void* stream,
           typename same_type<Args>::type... args) {
    return launch_resident(0, kernel, blocks, stream, args...);
}

struct SyncArgs {
    void* params;
    void* mom;          // fp32 or bf16 rows (Mom)
    float* mom2;
    const void* grads;  // fp32 or bf16 rows (Grad)
    float* slow;
    float* anchor;
    int W;
    int64_t P, ld;
    float beta, alpha;
    unsigned flags;
    void* stream;
};

}  // namespace
}  // namespace cpdp
