// The AllReduce calls of the C ABI: argument checks, and which form runs a call.
#include <cstdint>

#include "calls.h"
#include "device.h"
#include "forms.h"
#include "plan.h"

namespace {

// Argument checks shared by every form; OK with *run = false for a valid call without work.
int check_call(void* buffers, int n, int64_t elems, int dtype, const trivance_plan_t* plan,
               void* workspace, int64_t workspace_bytes, int pass_begin, int pass_end, bool* run) {
    *run = false;
    if (!plan || n != plan->n || elems < 0) return TRIVANCE_EINVAL;
    if (dtype != TRIVANCE_F32 && dtype != TRIVANCE_I32) return TRIVANCE_EINVAL;
    const int np = (int)plan->passes.size();
    if (pass_begin < 0 || pass_end < pass_begin || pass_end > np) return TRIVANCE_EINVAL;
    if (plan->variant == TRIVANCE_BRUCK_REF) return TRIVANCE_EUNSUPPORTED;
    if (elems == 0 || pass_begin == pass_end) return TRIVANCE_OK;
    if (!buffers) return TRIVANCE_EINVAL;
    const int64_t need = trivance_workspace_bytes(plan, elems, dtype);
    if (workspace_bytes < need || (need > 0 && !workspace)) return TRIVANCE_ESIZE;
    *run = true;
    return TRIVANCE_OK;
}

template <typename T>
int run_whole(T* buf, int64_t elems, const trivance_plan_t* plan, T* ws, hipStream_t stream) {
    switch (trivance::whole_form(plan, elems, (uintptr_t)buf % 16 == 0)) {
        case trivance::Form::kTile: return trivance::run_tile_call(buf, elems, plan, stream);
        case trivance::Form::kFold: return trivance::run_fold_call(buf, elems, plan, stream);
        case trivance::Form::kSweep: return trivance::run_sweep_call(buf, elems, plan, stream);
        default: break;
    }
    return trivance::run_step_passes(buf, elems, plan, ws, stream, 0, (int)plan->passes.size());
}

}  // namespace

extern "C" {

int64_t trivance_workspace_bytes(const trivance_plan_t* plan, int64_t elems, int dtype) {
    if (!plan || elems < 0) return TRIVANCE_EINVAL;
    if (dtype != TRIVANCE_F32 && dtype != TRIVANCE_I32) return TRIVANCE_EINVAL;
    if (plan->slots.empty()) return 0;
    return (int64_t)trivance::slot_halves(plan) * plan->max_slots * plan->n * elems * 4;
}

int trivance_allreduce_emulated_steps_ws(void* buffers, int n, int64_t elems, int dtype,
                                         const trivance_plan_t* plan, void* workspace,
                                         int64_t workspace_bytes, void* stream, int pass_begin,
                                         int pass_end) {
    bool run;
    const int rc = check_call(buffers, n, elems, dtype, plan, workspace, workspace_bytes, pass_begin,
                              pass_end, &run);
    if (!run) return rc;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (dtype == TRIVANCE_F32)
        return trivance::run_step_passes(static_cast<float*>(buffers), elems, plan,
                                         static_cast<float*>(workspace), s, pass_begin, pass_end);
    return trivance::run_step_passes(static_cast<int*>(buffers), elems, plan,
                                     static_cast<int*>(workspace), s, pass_begin, pass_end);
}

int trivance_allreduce_emulated_ws(void* buffers, int n, int64_t elems, int dtype,
                                   const trivance_plan_t* plan, void* workspace,
                                   int64_t workspace_bytes, void* stream) {
    if (!plan) return TRIVANCE_EINVAL;
    bool run;
    const int rc = check_call(buffers, n, elems, dtype, plan, workspace, workspace_bytes, 0,
                              (int)plan->passes.size(), &run);
    if (!run) return rc;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (dtype == TRIVANCE_F32)
        return run_whole(static_cast<float*>(buffers), elems, plan, static_cast<float*>(workspace), s);
    return run_whole(static_cast<int*>(buffers), elems, plan, static_cast<int*>(workspace), s);
}

int trivance_allreduce_emulated_steps(void* buffers, int n, int64_t elems, int dtype,
                                      const trivance_plan_t* plan, void* stream, int pass_begin,
                                      int pass_end) {
    return trivance_allreduce_emulated_steps_ws(buffers, n, elems, dtype, plan, nullptr, 0, stream,
                                                pass_begin, pass_end);
}

int trivance_allreduce_emulated(void* buffers, int n, int64_t elems, int dtype,
                                const trivance_plan_t* plan, void* stream) {
    return trivance_allreduce_emulated_ws(buffers, n, elems, dtype, plan, nullptr, 0, stream);
}

}  // extern "C"
