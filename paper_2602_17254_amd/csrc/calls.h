// The ways an AllReduce call can run, each in a source file of its own.
#pragma once

#include <hip/hip_runtime_api.h>

#include <cstdint>

#include "plan.h"

namespace trivance {

// Passes [pb, pe), one launch (or a few) per step (executor.hip, slot.hip). ws: the workspace of
// plans that keep partial sums.
int run_step_passes(float* buf, int64_t elems, const trivance_plan_t* p, float* ws,
                    hipStream_t stream, int pb, int pe);
int run_step_passes(int* buf, int64_t elems, const trivance_plan_t* p, int* ws, hipStream_t stream,
                    int pb, int pe);

// Whole bandwidth-optimal calls, each vector read once and written once (fold.hip). Which plans and sizes
// these and the forms below take: whole_form (forms.h).
int run_fold_call(float* buf, int64_t elems, const trivance_plan_t* p, hipStream_t stream);
int run_fold_call(int* buf, int64_t elems, const trivance_plan_t* p, hipStream_t stream);

// Small ones of these in tiles of local memory (tile.hip).
int run_tile_call(float* buf, int64_t elems, const trivance_plan_t* p, hipStream_t stream);
int run_tile_call(int* buf, int64_t elems, const trivance_plan_t* p, hipStream_t stream);

// The same for whole latency-optimal calls (sweep.hip).
int run_sweep_call(float* buf, int64_t elems, const trivance_plan_t* p, hipStream_t stream);
int run_sweep_call(int* buf, int64_t elems, const trivance_plan_t* p, hipStream_t stream);

}  // namespace trivance
