// gfx950 kernels: the later launches of the in-place update of tensors whose storage size changes
// (2 <-> 4 bytes per element), and the stand-alone conversion utility.
#include "resize_body.h"

namespace triaccel {

// Launches 1 .. n_stages - 1 of the in-place resize (launch 0 is part of the update kernel's grid).
template <bool ELEM, bool MOM>
__global__ __launch_bounds__(kThreads) void k_update_resize(const StepTables* __restrict__ tab, const TensorDesc* __restrict__ tds,
                                                            const GlobalDev* glob, StepScalars arg, uint32_t launch, uint32_t slots,
                                                            uint32_t n_wg) {
  const StepScalars sc = step_scalars(arg, *tab);
  // nothing to do on most steps: the two words that say so are read together
  const uint64_t skip_epoch = glob->skip_epoch;
  const uint32_t count = glob->trans_count[sc.step_id & 1u];
  TA_LOADED("s"(skip_epoch), "s"(count));
  if (count == 0 || skip_epoch == sc.step_id) return;
  resize_items<ELEM, MOM>(*tab, tds, count, launch, slots, blockIdx.x, n_wg, sc);
}

// ---------------------------------------------------------------------------------------------
// Utility: fp32 -> {fp16, bf16, fp32} array conversion with the store path of the update kernel.
// ---------------------------------------------------------------------------------------------
template <int ND>
__global__ __launch_bounds__(kThreads) void k_cast(const float* __restrict__ src, void* dst, int64_t n) {
  // same shape as the step kernels: one workgroup per chunk, all loads of the chunk before its stores
  const int64_t base = (int64_t)blockIdx.x * kChunk;
  const int32_t left = chunk_left(base, n);
  constexpr int W = kWords<ND>;
  uint32_t w[kRows][4];
  const Tail tail = tail_of(left, threadIdx.x);
  const uint32_t wt = load_chunk<4>(src + base, left, tail, w);
  void* const to = chunk_of<W>(dst, base);
  const Rows rows = rows_of<W>(to, left);
#pragma unroll
  for (int r = 0; r < kRows; ++r) {
    narrow4<ND>(w[r]);
    store_words<W>(rows, r, threadIdx.x, w[r]);
  }
  if (tail.any) store_tail<ND>(to, tail, wt);
}

hipError_t launch_update_resize(const DeviceTables& t, const StepScalars& sc, bool elem, hipStream_t s) {
  const bool mom = t.hyper.momentum != 0.0f;
  const auto kernel = elem ? (mom ? k_update_resize<true, true> : k_update_resize<true, false>)
                           : (mom ? k_update_resize<false, true> : k_update_resize<false, false>);
  for (uint32_t q = 1; q < t.plan.n_stages; ++q) {
    const ResizeGrid rg = resize_grid(t.plan, q, t.n_tensors, t.total_chunks < kResizeBigSet);
    const hipError_t e = launch(kernel, rg.grid, kThreads, s, t.dev, t.tensors, t.glob, sc, q, rg.slots, rg.grid);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

__global__ void k_set_scalars(StepScalars v, StepScalars* dst) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *dst = v;
}

hipError_t launch_set_scalars(const DeviceTables& t, const StepScalars& sc, hipStream_t s) {
  return launch(k_set_scalars, 1, kWave, s, sc, &t.dev->scalars);
}

void set_scalars_node_params(hipKernelNodeParams* p, void** args, const StepScalars* sc, StepScalars* const* dst) {
  args[0] = const_cast<StepScalars*>(sc);
  args[1] = const_cast<StepScalars**>(dst);
  p->func = reinterpret_cast<void*>(k_set_scalars);
  p->gridDim = dim3(1);
  p->blockDim = dim3(kWave);
  p->sharedMemBytes = 0;
  p->kernelParams = args;
  p->extra = nullptr;
}

hipError_t launch_cast(const float* src, void* dst, int64_t n, int dtype, hipStream_t s) {
  int64_t blocks = (n + kChunk - 1) / kChunk;
  if (blocks < 1) blocks = 1;
  const auto kernel = dtype == kFP32 ? k_cast<kFP32> : dtype == kBF16 ? k_cast<kBF16> : k_cast<kFP16>;
  return launch(kernel, (uint32_t)blocks, kThreads, s, src, dst, n);
}

}  // namespace triaccel
