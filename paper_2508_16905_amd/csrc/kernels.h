// Host-callable launchers of the gfx950 kernels (defined in kernels.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "common.h"
#include "resize_schedule.h"

namespace triaccel {

// A pointer into device memory that kernels read from memory themselves.  They have to know that it is a global one: of
// any other they make FLAT accesses (numerics.h), with a 64-bit address per lane and never through the scalar caches.
template <typename T>
struct DevPtr {
#if defined(__HIP_DEVICE_COMPILE__)
  __attribute__((address_space(1))) T* p;
#else
  T* p;
#endif
  __host__ __device__ operator T*() const { return (T*)p; }
};

// What the step's kernels know of a handle beyond their arguments: pointers into its workspace, its configuration and
// sizes, constant from triaccel_init on and kept in device memory.  A launch costs the host 2.6 us with up to 64 bytes of
// arguments, 3.2 with 128, 3.5 with 330 and 4.1 if those are 20 separate ones and the hidden ones of a kernel that asks for
// its grid's size, and that is what sets bound by their launches wait for.  So the kernels get the pointers that their
// first loads need (this one, the tensor table, the chunk list, the global record), the step's scalars and up to four
// words more; the loads from here go beside those of the chunk's and the tensor's entries, so that no access to the
// data comes later for them.  A step, us, with up to 20 arguments and now (the latter with the
// pointers preloaded, build.py): two-layer perceptron 10.2 and 8.0, with a probe, fp16 gradients and the result read 28.2 and
// 26.7; 12 tensors of 2000 elements in all with a probe 14.9 and 11.9; 41 of 1.0 M with step sizes per element 37.4 and
// 34.0; EfficientNet-B0 set, bf16, 16.0 and 14.9, ResNet-18 set 43.0 and 42.9.
struct StepTables {
  StepScalars scalars;          // of a replayed graph's step, written by its first kernel
  DevPtr<ChunkRef> chunks;      // tensor by tensor, in order; then the order heads_first, in sets that use it
  DevPtr<StatPartial> partials; // one record per chunk, in the order of `chunks`
  DevPtr<EmaPartial> ema_partials;  // the same, written by the EMA kernel
  DevPtr<LayerDev> layers;
  DevPtr<GlobalDev> host_result;    // pinned host memory (device-visible address): the step's result record
  DevPtr<uint32_t> hist;            // n_tensors x kHistBins
  DevPtr<Candidate> cands;          // pool of the tensors' key lists (key_lists)
  DevPtr<uint32_t> cand_counters;   // n_tensors x (kCandLists + 1) counters, kCandCounterStride words apart
  DevPtr<uint32_t> trans_list;      // 2 x n_tensors
  DevPtr<char> resize_scratch;  // new values of the first chunks of tensors that change size (resize_schedule.h)
  DevPtr<LayerIn> inputs;       // n_tensors: what the running step's decisions read of the layers' records (k_update_local)
  DevPtr<uint32_t> arrived;     // n_tensors counters, kCandCounterStride words apart: chunks done in a fallback pass; 0 between steps
  DevPtr<float> undo_h;         // curvature and mask words that a step overwrites before it is known to be taken (kFusedChunks)
  DevPtr<uint32_t> undo_mask;
  uint32_t n_tensors;
  uint32_t total_chunks;
  Hyper hyper;
  ResizePlan plan;
};

// A handle's workspace as the launchers see it.
struct DeviceTables : StepTables {
  StepTables* dev;           // the device copy of the part above; graphs write its scalars
  TensorDesc* tensors;
  const ChunkRef* wg_chunks; // chunk of each workgroup of the kernels that have one for every chunk: `chunks`, or heads_first
  GlobalDev* glob;
  uint32_t max_chunks_per_tensor;
  bool all_small;            // no tensor is longer than kListAllMax: their keys always settle the thresholds
  bool fused;                // probed steps take statistics and curvature in one launch, and have the workspace for it
  bool keep_grads;           // the gradients of the set have at most kKeepBytes
  uint32_t persistent_grid;  // workgroups of the persistent streaming kernels
};

hipError_t launch_grad_stats(const DeviceTables& t, const StepScalars& sc, bool local, hipStream_t s);
hipError_t launch_curv_ema(const DeviceTables& t, const StepScalars& sc, bool fisher, bool local, hipStream_t s);
// Both of these, on probed steps of sets that have the workspace for it (`fused`).
hipError_t launch_stats_ema(const DeviceTables& t, const StepScalars& sc, bool fisher, hipStream_t s);
hipError_t launch_hist_pass(const DeviceTables& t, const StepScalars& sc, int serial_rounds, hipStream_t s);
hipError_t launch_select_finish(const DeviceTables& t, const StepScalars& sc, hipStream_t s);
hipError_t launch_layer(const DeviceTables& t, const StepScalars& sc, hipStream_t s);
// `resize`: with launch 0 of the in-place resize.
hipError_t launch_update(const DeviceTables& t, const StepScalars& sc, bool elem, bool resize, hipStream_t s);
// `undo`: after k_stats_ema.
hipError_t launch_update_local(const DeviceTables& t, const StepScalars& sc, bool any_probe, bool undo, hipStream_t s);
// Probed steps with step sizes per element, on sets within kDecideMaxChunks and kDecideTotalChunks: the layers' decisions and most
// thresholds.
hipError_t launch_decide_select(const DeviceTables& t, const StepScalars& sc, bool undo, hipStream_t s);
// `local`: after k_update_local or k_decide_select, which settled most tensors' thresholds; `resize`: with launch 1 of the
// in-place resize (sets of the local form: its plans have two launches at most).
hipError_t launch_select_tail(const DeviceTables& t, const StepScalars& sc, bool local, bool resize, hipStream_t s);
hipError_t launch_mask_pass(const DeviceTables& t, const StepScalars& sc, hipStream_t s);
hipError_t launch_update_resize(const DeviceTables& t, const StepScalars& sc, bool elem, hipStream_t s);
// Writes the per-step scalars to device memory (first node of a captured step).
hipError_t launch_set_scalars(const DeviceTables& t, const StepScalars& sc, hipStream_t s);
// Kernel-node parameters of that launch, for updating an instantiated graph; `args` must hold two
// pointers and outlive the call that consumes the parameters.
void set_scalars_node_params(hipKernelNodeParams* p, void** args, const StepScalars* sc, StepScalars* const* dst);
hipError_t launch_cast(const float* src, void* dst, int64_t n, int dtype, hipStream_t s);

// One launch on `s`: hipLaunchKernel without the call-configuration stack of <<<>>> (0.1 us).
template <typename... P, typename... A>
hipError_t launch(void (*kernel)(P...), uint32_t grid, uint32_t threads, hipStream_t s, A... a) {
  static_assert(sizeof...(P) == sizeof...(A), "one argument per parameter");
  return [&](P... p) {
    void* args[] = {static_cast<void*>(&p)...};
    return hipLaunchKernel(reinterpret_cast<const void*>(kernel), dim3(grid), dim3(threads), args, 0, s);
  }(a...);
}

}  // namespace triaccel
