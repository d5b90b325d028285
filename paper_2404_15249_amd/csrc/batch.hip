// Batched KFBI steps: many problems of uneven size advance through one launch
// per stage of a GMRES iteration.  Every launch is persistent: a fixed grid
// walks a device-resident work list of (slot, block) items, so the same
// recorded graph serves any mix of live slots, and a slot that has converged
// turns its items into no-ops.  Each slot's arithmetic is split into the same
// blocks whatever else is in the batch (one workgroup partial per mode block,
// fixed reduction order), so its result does not depend on the mix.
#include <hip/hip_runtime.h>

#include "batch.h"
#include "device.h"
#include "gmres.h"
#include "graph.h"

namespace kfbi {

namespace {

__device__ __forceinline__ bool slot_done(const SlotDev& S) { return S.b.st->converged != 0; }

template <int C>
__device__ __forceinline__ void modes_item(const DevPlan& p, const double* corr, int row, const ModesLds& L,
                                           double* part) {
    constexpr int R = batch_modes_per_group(64 * C);
    modes_round<C, R, false, false>(p, corr, row, L, [&](int, int cp, double s) { part[(size_t)row * p.M + cp] = s; });
}

__global__ __launch_bounds__(kModeWaves * 64) void k_modes_b(const SlotDev* __restrict__ slots, BatchWork w) {
    extern __shared__ double smem[];
    ModesLds L;
    L.sq = smem;
    L.xs = smem + kBatchTable;
    static_assert(kBatchModes == 0, "the first list");
    const int n_items = w.counts[1];
    for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
        const int2 item = w.items[it];
        const SlotDev& S = slots[item.x];
        if (S.b.st->skip) continue;
        const DevPlan& p = S.p;
        switch (p.N) {
            case 64: modes_item<1>(p, S.corr_il, item.y, L, S.partial); break;
            case 128: modes_item<2>(p, S.corr_il, item.y, L, S.partial); break;
            case 256: modes_item<4>(p, S.corr_il, item.y, L, S.partial); break;
            case 512: modes_item<8>(p, S.corr_il, item.y, L, S.partial); break;
            case 1024: modes_item<16>(p, S.corr_il, item.y, L, S.partial); break;
            case 2048: modes_item<32>(p, S.corr_il, item.y, L, S.partial); break;
            default: modes_item<64>(p, S.corr_il, item.y, L, S.partial); break;
        }
    }
}

// A slot's reduce items: 64 samples from item.y on, or (item.y < 0) its commit.
__global__ __launch_bounds__(1024) void k_reduce_b(BatchWork w) {
    __shared__ double red[16 * 64];
    const int n_items = w.counts[kBatchReduce + 1];
    for (int it = w.counts[kBatchReduce] + blockIdx.x; it < n_items; it += gridDim.x) {
        const int2 item = w.items[it];
        const SlotDev& S = w.slots[item.x];
        if (item.y < 0) {
            gm_commit(S.b, S.p.M);
        } else if (!slot_done(S)) {
            const GmPre<1> pre = gm_reduce_prefetch(S.b, S.p.M, item.y / 64);
            const GmPh ph{S.b.st->ph, S.b.st->j, S.b.st->second, S.b.st->reorth};
            const JumpSrc js{S.b.xcur, S.b.s2cur, nullptr, nullptr, nullptr, nullptr};
            reduce_samples64(S.p, js, S.partial, S.Gs, item.y, nullptr, red);
            gm_reduce64(S.b, S.p.M, item.y / 64, red, pre, ph);
        }
        __syncthreads();                                 // the item's LDS is reused by the next item
    }
}

// GMRES (gmres.h): the step launch walks (slot, chunk) items, the vector's chunks
// and then the correction chunks of each slot.
__global__ __launch_bounds__(kGmChunk) void k_gm_step_b(BatchWork w) {
    const int n_items = w.counts[kBatchSteps + 1];
    for (int it = w.counts[kBatchSteps] + blockIdx.x; it < n_items; it += gridDim.x) {
        const int2 item = w.items[it];
        const SlotDev& S = w.slots[item.x];
        if (item.y < S.b.gc) {
            gm_step(S.p.taps, S.b, S.p.M, item.y);
        } else {
            gm_step_corrections(S.p, S.b, item.y - S.b.gc, S.corr_il);
        }
        __syncthreads();                                 // the item's LDS is reused by the next item
    }
}

// The poll's states, together: a copy for each slot took 3 us of the stream and more of
// the host (twelve of them four times were a fifth of a batch of 12).
__global__ __launch_bounds__(64) void k_states_b(BatchWork w, int max_slots, GmresState* __restrict__ out) {
    const int k = blockIdx.x * 64 + threadIdx.x;
    if (k < max_slots && w.slots[k].live) out[k] = *w.slots[k].b.st;
}

}  // namespace

size_t modes_b_lds_bytes() {
    return sizeof(double) * ((size_t)kBatchTable + (size_t)kBatchXs);
}

hipError_t launch_batch_step(BatchWork w, int n_cu, hipStream_t s) {
    const size_t lds = modes_b_lds_bytes();
    if (hipError_t e = hipFuncSetAttribute((const void*)k_modes_b, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds))
        return e;
    if (hipError_t e = klaunch(&k_modes_b, dim3(n_cu), dim3(kModeWaves * 64), lds, s, w.slots, w)) return e;
    if (hipError_t e = klaunch(&k_reduce_b, dim3(n_cu), dim3(1024), 0, s, w)) return e;
    return klaunch(&k_gm_step_b, dim3(n_cu), dim3(kGmChunk), 0, s, w);
}

hipError_t launch_batch_states(BatchWork w, int max_slots, GmresState* out, hipStream_t s) {
    return klaunch(&k_states_b, dim3((max_slots + 63) / 64), dim3(64), 0, s, w, max_slots, out);
}

}  // namespace kfbi
