// Device descriptors of the batched KFBI steps (see batch.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.h"

namespace kfbi {

constexpr int kBatchNmax = 4096;    // largest grid a batch serves
// LDS of the batched fast solve holds this many doubles of mode solutions and sums
// of extra pieces: eight modes of the 2048^2 grid, four of the 4096^2 grid
constexpr int kBatchXs = 4 * (2 * modes_stride_of(2048) + kMaxExtra);
constexpr int kBatchTable = 96 * 32 + 4;   // the largest table of sines and cosines (modes_table_len at 2048)

// Modes per workgroup of a batched problem with grid N: the largest power of two
// up to kMaxModesPerGroup whose padded solutions fit kBatchXs.
__host__ __device__ constexpr int batch_modes_per_group(int N) {
    int R = kMaxModesPerGroup;
    while (R > 2 && R / 2 * (2 * modes_stride_of(N) + kMaxExtra) > kBatchXs) R /= 2;
    return R;
}

// One live problem of a batch, resident in device memory.
struct SlotDev {
    DevPlan p;
    GmresBufs b;
    double* corr_il;   // interleaved corrections (T x 64)
    double* partial;   // Gs x M partial sums, one row per mode block
    int Gs;            // mode blocks: ceil((n-1) / batch_modes_per_group(N))
    int live;          // the slot holds a problem
};

// Work lists of the batched launches, rebuilt on the host when a slot is admitted or
// released: (slot, first index) pairs, one list after the other in items, list k from
// counts[k] up to counts[k + 1]:
enum BatchList {
    kBatchModes = 0,    // mode blocks of batch_modes_per_group(N) modes, the largest grids first
    kBatchReduce = 1,   // blocks of 64 samples, and (slot, -1) the commit
    kBatchSteps = 2,    // (slot, chunk): vector chunks, then correction chunks
    kBatchLists = 3
};
// The counts, the slots and the items are one allocation and one upload: an admission
// or a release copied five arrays before, 3 us of the stream each.
struct BatchWork {
    const int* counts;        // kBatchLists + 1
    const SlotDev* slots;
    const int2* items;
};

size_t modes_b_lds_bytes();
hipError_t launch_batch_step(BatchWork w, int n_cu, hipStream_t s);
// out[k] <- the GMRES state of slot k, live slots only
hipError_t launch_batch_states(BatchWork w, int max_slots, GmresState* out, hipStream_t s);

}  // namespace kfbi
