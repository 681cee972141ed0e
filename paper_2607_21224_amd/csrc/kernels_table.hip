// Step tables: the local and synchronisation steps with their scalars read
// from a device table, and the kernels that move the table's position.
#include "cpdp_split.h"

namespace cpdp {
namespace {

// J <= kMaxLocalSteps consecutive local steps of one replica's 4 coordinates,
// step j with gradient rows g.rows[j] and the entry ahead + j places past the
// position.  A local step touches only its own coordinates, so the steps in
// between need not go through memory: the state is read and written once and
// all gradients are in flight together (3 AdamW steps of 8 x 100,003 in one
// captured graph, without the advances: 3 x 5.0 us before, 9.4 in one).  bf16
// parameters are rounded after every step, as a store and a load would.
struct GradRows {
    const float* rows[kMaxLocalSteps];
};

template <Opt O, class PS, int F>
__device__ __forceinline__ void local_steps_chunk(const int64_t* table, int64_t ahead,
                                                  const GradRows& gr, int J,
                                                  typename PS::T* params, float* mom, float* mom2,
                                                  int64_t at, int n) {
    float g[kMaxLocalSteps][kVec], m[kVec], v[kVec], th[kVec];
    load_f32<F, kNTL>(mom + at, n, m);
    if constexpr (O == Opt::ADAMW) load_f32<F, kNTL>(mom2 + at, n, v);
    PS::template load<F, kNTL>(params + at, n, th);
#pragma unroll
    for (int j = 0; j < kMaxLocalSteps; ++j)
        if (j < J) load_f32<F, kNTL>(gr.rows[j] + at, n, g[j]);
    loads_first();
    StepEntry e;
    if (!step_entry(table, ahead, e)) return;
#pragma unroll
    for (int j = 0; j < kMaxLocalSteps; ++j) {
        // the state stays as it is once the table is used up
        if (j >= J || (j > 0 && !step_entry(table, ahead + j, e))) break;
#pragma unroll
        for (int k = 0; k < kVec; ++k) th[k] = opt_update<O, PS>(e.o, th[k], m[k], v[k], g[j][k]);
    }
    store_f32<F, kNTS>(mom + at, n, m);
    if constexpr (O == Opt::ADAMW) store_f32<F, kNTS>(mom2 + at, n, v);
    PS::template store<F, kNTS>(params + at, n, th);
}

template <Opt O, class PS>
__global__ __launch_bounds__(kBlock) void local_steps_table_kernel(
    const int64_t* table, int64_t ahead, typename PS::T* params, float* mom, float* mom2,
    GradRows grads, int J, int64_t ld, int64_t P, int64_t blocks_per_row, int64_t cells) {
    const int64_t cell = local_cell(cells);
    if (cell < 0) return;
    const int64_t row = cell / blocks_per_row;
    const int64_t col = cell - row * blocks_per_row;
    const int64_t p0 = (col * kBlock + threadIdx.x) * kVec;
    if (p0 >= P) return;
    for_lanes(p0, P, [&](auto lanes, int n) {
        local_steps_chunk<O, PS, lanes>(table, ahead, grads, J, params, mom, mom2, row * ld + p0,
                                        n);
    });
}

// run-time W (replica batches of kChunk): one instantiation per strategy,
// update and parameter type, whatever W is
template <Sync M, Opt O, class PS, bool EXTRA>
__global__ __launch_bounds__(kBlock) void sync_table_kernel(
    const int64_t* __restrict__ table, int64_t ahead, typename PS::T* __restrict__ params,
    float* __restrict__ mom, float* __restrict__ mom2, GradPtr<EXTRA> __restrict__ grads,
    float* __restrict__ slow, float* __restrict__ anchor, int W, int64_t ld, int64_t P,
    float inv_w, unsigned flags) {
    const int64_t p0 = ((int64_t)blockIdx.x * kBlock + threadIdx.x) * kVec;
    if (p0 >= P) return;
    StepEntry e;
    if (!step_entry(table, ahead, e)) return;
    const Strided<PS> r{params, mom, mom2, const_cast<float*>(grads), ld};
    for_lanes(p0, P, [&](auto lanes, int n) {
        sync_chunk<M, O, 0, PS, lanes, EXTRA>(e.o, r, slow, anchor, W, p0, n, e.beta, e.alpha_lr,
                                              inv_w, flags);
    });
}

// position word updates: one lane of one block, an ordinary (vector) store
__global__ __launch_bounds__(64) void step_table_set_kernel(int64_t* table, int64_t position) {
    if (blockIdx.x == 0 && threadIdx.x == 0) table[0] = position;
}

__global__ __launch_bounds__(64) void step_table_advance_kernel(int64_t* table, int64_t steps) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        const int64_t pos = table[0], left = table[1] - pos;
        if (left > 0) table[0] = pos + min(steps, left);
    }
}

template <Opt O>
int local_table_o(Param pt, const int64_t* table, int64_t ahead, void* params, float* mom,
                  float* mom2, const GradRows& grads, int J, int W, int64_t P, int64_t ld,
                  void* stream) {
    const int64_t bpr = blocks_for(P);
    if (pt == Param::BF16)
        return launch(local_steps_table_kernel<O, ParamBF16>, local_grid(bpr * W), stream, table,
                      ahead, static_cast<uint16_t*>(params), mom, mom2, grads, J, ld, P, bpr,
                      bpr * W);
    return launch(local_steps_table_kernel<O, ParamF32>, local_grid(bpr * W), stream, table,
                  ahead, static_cast<float*>(params), mom, mom2, grads, J, ld, P, bpr, bpr * W);
}

template <Sync M, Opt O, class PS>
int sync_table_t(const TableScalars& src, const SyncArgs& a) {
    using T = typename PS::T;
    const float inv_w = 1.0f / (float)a.W;
    if (can_split(a.W, blocks_for(a.P), kBlock) &&
        !takes_columns(step_kind<M, O, PS>(), a.W, a.P, true)) {
        return a.flags != 0 ? sync_split<M, O, PS, true, ParamF32, ParamF32>(src, a)
                            : sync_split<M, O, PS, false, ParamF32, ParamF32>(src, a);
    }
    // step tables take fp32 gradients
    const float* grads = static_cast<const float*>(a.grads);
    const int resident = run_time_waves(step_kind<M, O, PS>(), a.W, a.P, RunTime::Table);
    if (a.flags != 0)
        return launch_resident(resident, sync_table_kernel<M, O, PS, true>, blocks_for(a.P),
                               a.stream, src.table, src.ahead, static_cast<T*>(a.params),
                               static_cast<float*>(a.mom), a.mom2, const_cast<float*>(grads),
                               a.slow, a.anchor, a.W, a.ld, a.P, inv_w, a.flags);
    return launch_resident(resident, sync_table_kernel<M, O, PS, false>, blocks_for(a.P),
                           a.stream, src.table, src.ahead, static_cast<T*>(a.params),
                           static_cast<float*>(a.mom), a.mom2, grads, a.slow, a.anchor, a.W, a.ld,
                           a.P, inv_w, a.flags);
}

template <Sync M, Opt O>
int sync_table_p(Param pt, const TableScalars& src, const SyncArgs& a) {
    return pt == Param::BF16 ? sync_table_t<M, O, ParamBF16>(src, a)
                             : sync_table_t<M, O, ParamF32>(src, a);
}

template <Sync M>
int sync_table_o(Opt opt, Param pt, const TableScalars& src, const SyncArgs& a) {
    switch (opt) {
        case Opt::SGD_WD: return sync_table_p<M, Opt::SGD_WD>(pt, src, a);
        case Opt::ADAMW: return sync_table_p<M, Opt::ADAMW>(pt, src, a);
        default: return sync_table_p<M, Opt::SGD>(pt, src, a);
    }
}

}  // namespace

int launch_local_steps_table(Opt opt, Param pt, const int64_t* table, int64_t ahead, void* params,
                             float* mom, float* mom2, const float* const* grads, int J, int W,
                             int64_t P, int64_t ld, void* stream) {
    GradRows g{};
    for (int j = 0; j < J; ++j) g.rows[j] = grads[j];
    switch (opt) {
        case Opt::SGD_WD:
            return local_table_o<Opt::SGD_WD>(pt, table, ahead, params, mom, mom2, g, J, W, P, ld,
                                              stream);
        case Opt::ADAMW:
            return local_table_o<Opt::ADAMW>(pt, table, ahead, params, mom, mom2, g, J, W, P, ld,
                                             stream);
        default:
            return local_table_o<Opt::SGD>(pt, table, ahead, params, mom, mom2, g, J, W, P, ld,
                                           stream);
    }
}

int launch_sync_table_ahead(Sync mode, Opt opt, Param pt, const int64_t* table, int64_t ahead,
                            void* params, float* mom, float* mom2, const float* grads, float* slow,
                            float* anchor, int W, int64_t P, int64_t ld, unsigned flags,
                            void* stream) {
    const SyncArgs a{params, mom, mom2, grads, slow, anchor, W, P, ld, 0.0f, 1.0f, flags, stream};
    const TableScalars src{table, ahead};
    switch (mode) {
        case Sync::LocalSGD: return sync_table_o<Sync::LocalSGD>(opt, pt, src, a);
        case Sync::DDP: return sync_table_o<Sync::DDP>(opt, pt, src, a);
        default: return sync_table_o<Sync::CPDP>(opt, pt, src, a);
    }
}

int launch_step_table_set(int64_t* table, int64_t position, void* stream) {
    void* argv[] = {static_cast<void*>(&table), static_cast<void*>(&position)};
    return (int)hipLaunchKernel(reinterpret_cast<const void*>(step_table_set_kernel), dim3(1),
                                dim3(64), argv, 0, static_cast<hipStream_t>(stream));
}

int launch_step_table_advance_by(int64_t* table, int64_t steps, void* stream) {
    void* argv[] = {static_cast<void*>(&table), static_cast<void*>(&steps)};
    return (int)hipLaunchKernel(reinterpret_cast<const void*>(step_table_advance_kernel), dim3(1),
                                dim3(64), argv, 0, static_cast<hipStream_t>(stream));
}

int read_step_table_position(const int64_t* table, int64_t* position) {
    return (int)hipMemcpy(position, table, sizeof(int64_t), hipMemcpyDeviceToHost);
}

int upload_bytes(void* dev, const void* host, int64_t bytes) {
    return (int)hipMemcpy(dev, host, (size_t)bytes, hipMemcpyHostToDevice);
}

}  // namespace cpdp
