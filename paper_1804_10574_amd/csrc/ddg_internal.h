// Calls shared by the module and the pipeline that are not part of the C boundary.
#pragma once
#include "../../include/ddg.h"
#include <hip/hip_runtime_api.h>

extern "C" {
// While set, the module's calls advance their host-side state (iteration counter, ring
// position) and validate arguments but enqueue nothing: the pipeline replays a captured
// graph of the same call instead.
void ddg_internal_skip_launches(ddg_module* m, bool skip);
// The update reads its step size from this device float instead of the call argument.
void ddg_internal_lr_from(ddg_module* m, const float* lr_dev);
bool ddg_internal_profiling(const ddg_module* m);
// What ddg_forward_eval refuses, without its launches.
ddg_status ddg_internal_eval_ok(ddg_module* m, const void* h_in, void* h_out, const int32_t* labels, float* loss_out);
// Evaluation passes of the module go to stream s (on) or to its own stream again (off).
void ddg_internal_eval_stream(ddg_module* m, bool on, hipStream_t s);
// A pipeline orders the module's two streams itself (events around graph launches); the module
// then records and waits on nothing.
void ddg_internal_external_sync(ddg_module* m, bool on);
// While on, ddg_backward_delayed may leave sums of weight gradients to the ddg_update that the caller issues right after it.
void ddg_internal_fuse_update(ddg_module* m, bool on);
// The streams ddg_forward and ddg_backward_delayed/ddg_update enqueue on (equal unless the
// module runs its forward pass on a stream of its own).
void ddg_internal_streams(ddg_module* m, hipStream_t* fwd, hipStream_t* bwd);
// Sets the message ddg_last_error returns on this thread.
void ddg_internal_set_error(const char* msg);
}
