// Host-callable launchers of the gfx950 kernels (defined in kernels.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "common.h"

namespace triaccel {

// Device pointers and sizes of a handle's workspace.
struct DeviceTables {
  TensorDesc* tensors;
  ChunkRef* chunks;          // tensor by tensor, in order; then the order heads_first, in sets that use it
  const ChunkRef* wg_chunks; // chunk of each workgroup of the kernels that have one for every chunk: `chunks`, or heads_first
  StatPartial* partials;     // one record per chunk, in the order of `chunks`
  EmaPartial* ema_partials;  // the same, written by the EMA kernel
  LayerDev* layers;
  GlobalDev* glob;
  GlobalDev* host_result;  // pinned host memory (device-visible address): the per-layer kernel leaves the step's result record there
  uint32_t* hist;        // n_tensors x kHistBins
  Candidate* cands;      // pool of the tensors' key lists (key_lists)
  uint32_t* cand_counters;  // n_tensors x (kCandLists + 1) counters, kCandCounterStride words apart
  uint32_t* trans_list;  // 2 x n_tensors
  char* resize_scratch;  // new values of the first chunks of tensors that change size (resize_schedule.h)
  LayerIn* inputs;       // n_tensors: what the running step's decisions read of the layers' records (k_update_local)
  uint32_t* arrived;     // n_tensors counters, kCandCounterStride words apart: chunks done in a fallback pass; 0 between steps
  StepScalars* scalars;  // device copy of the per-step scalars, read by the kernels of a replayed graph
  uint32_t n_tensors;
  uint32_t total_chunks;
  uint32_t max_chunks_per_tensor;
  bool all_small;            // no tensor is longer than kListAllMax: their keys always settle the thresholds
  bool keep_grads;           // the gradients of the set have at most kKeepBytes
  uint32_t persistent_grid;  // workgroups of the persistent streaming kernels
};

hipError_t launch_grad_stats(const DeviceTables& t, const StepArg& sa, bool local, hipStream_t s);
hipError_t launch_curv_ema(const DeviceTables& t, const StepArg& sa, float beta_h, float omb_h, int fisher, bool local,
                           hipStream_t s);
hipError_t launch_hist_pass(const DeviceTables& t, const StepArg& sa, int serial_rounds, hipStream_t s);
hipError_t launch_select_finish(const DeviceTables& t, const StepArg& sa, float beta_h, hipStream_t s);
hipError_t launch_layer(const DeviceTables& t, const StepArg& sa, const Hyper& hp, hipStream_t s);
// `resize`: with launch 0 of the in-place resize.
hipError_t launch_update(const DeviceTables& t, const StepArg& sa, float wd, float mu, float alpha, bool elem, bool resize,
                         hipStream_t s);
hipError_t launch_update_local(const DeviceTables& t, const StepArg& sa, const Hyper& hp, bool any_probe, hipStream_t s);
// `local`: after k_update_local, which settled most tensors' thresholds; `resize`: with launch 1 of the in-place resize (sets
// of the local form: its plans have two launches at most).
hipError_t launch_select_tail(const DeviceTables& t, const StepArg& sa, const Hyper& hp, bool local, bool resize, hipStream_t s);
hipError_t launch_mask_pass(const DeviceTables& t, const StepArg& sa, hipStream_t s);
hipError_t launch_update_resize(const DeviceTables& t, const StepArg& sa, float wd, float mu, float alpha,
                                bool elem, hipStream_t s);
// Writes the per-step scalars to device memory (first node of a captured step).
hipError_t launch_set_scalars(const DeviceTables& t, const StepScalars& sc, hipStream_t s);
// Kernel-node parameters of that launch, for updating an instantiated graph; `args` must hold two
// pointers and outlive the call that consumes the parameters.
void set_scalars_node_params(hipKernelNodeParams* p, void** args, const StepScalars* sc, StepScalars* const* dst);
hipError_t launch_cast(const float* src, void* dst, int64_t n, int dtype, hipStream_t s);

}  // namespace triaccel
