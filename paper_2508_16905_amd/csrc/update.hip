// gfx950 kernels of the fused update + cast (stage 5 of the optimizer step) and the stand-alone
// mask pass.  Compiled as a translation unit of its own: the update body is specialised for every
// (gradient, old, new) precision triple, which dominates the build time.
#include "resize_body.h"

namespace triaccel {

// Mask pass as a kernel of its own, for the element-wise form of the update, where the threshold
// must be final before the update runs: the tensors whose mask the EMA kernel did not settle get
// their mask written and their range keys listed here, before k_select_finish.  Leaves at once
// when no tensor needs it (the steady state).
__global__ __launch_bounds__(kThreads) void k_mask_pass(const StepTables* __restrict__ tab, const TensorDesc* __restrict__ tds,
                                                        const ChunkRef* __restrict__ chunks, const GlobalDev* glob, StepScalars arg,
                                                        uint32_t n_wg) {
  const StepScalars sc = step_scalars(arg, *tab);
  const LayerDev* const layers = tab->layers;
  const uint32_t total_chunks = tab->total_chunks;
  const uint64_t skip_epoch = glob->skip_epoch;
  const uint32_t pending = glob->mask_pending[sc.step_id & 1u];
  TA_LOADED("s"(skip_epoch), "s"(pending));
  if (pending == 0 || skip_epoch == sc.step_id) return;
  for (uint32_t c = blockIdx.x; c < total_chunks; c += n_wg) {
    const ChunkRef cr = chunks[c];
    const TensorDesc td = tds[cr.tensor];
    const LayerDev& ls = layers[cr.tensor];
    const uint32_t mode = ls.mode;
    if (!td.has_probe || ls.mask_done || mode == kSelHist) continue;
    const int64_t base = (int64_t)cr.index * kChunk;
    mask_chunk(td, base, mode, ls.theta_key, ls.rng_lo, ls.rng_hi, cr.index, cr.tensor, tab->cands, tab->cand_counters);
  }
}

// Tensors whose storage size does not change: element i is read and written at the same address
// by the same lane, so the update is in place.  One workgroup per chunk.  The same workgroup then
// runs the fallback mask pass of its chunk when the tensor's mask was not settled by the EMA
// kernel (nothing in the update depends on the mask, and a separate launch would cost a full
// grid of idle workgroups on every step that needs no fallback).
//
// The first `resize_wgs` workgroups of the grid do something else: the first launch of the in-place
// resize of the tensors whose storage size does change (resize_body.h).  It depends on the per-layer
// kernel only, like the update itself, so it needs no launch of its own; it comes first in the grid
// because its work items are the longer ones.
//
// In the element-wise form (ELEM) the threshold must be final before the update, so the mask and
// the listed keys are completed by the kernels before this one and no mask pass runs here.
template <bool ELEM, bool MOM>
__global__ __launch_bounds__(kThreads) void k_update(const StepTables* __restrict__ tab, const TensorDesc* __restrict__ tds,
                                                     const ChunkRef* __restrict__ chunks, const GlobalDev* glob, StepScalars arg,
                                                     uint32_t resize_slots, uint32_t resize_wgs) {
  const StepScalars sc = step_scalars(arg, *tab);
  const LayerDev* const layers = tab->layers;
  const float wd = tab->hyper.weight_decay, mu = tab->hyper.momentum, alpha = tab->hyper.alpha;
  if (blockIdx.x < resize_wgs) {
    const uint64_t skip_epoch = glob->skip_epoch;
    const uint32_t count = glob->trans_count[sc.step_id & 1u];
    TA_LOADED("s"(skip_epoch), "s"(count));
    if (count == 0 || skip_epoch == sc.step_id) return;
    resize_items<ELEM, MOM>(*tab, tds, count, 0u, resize_slots, blockIdx.x, resize_wgs, sc);
    return;
  }
  // the skip word travels together with the tables: its latency is not one more before the data's
  const uint64_t skip_epoch = glob->skip_epoch;
  const ChunkRef cr = chunks[blockIdx.x - resize_wgs];
  const LayerDev& ls = layers[cr.tensor];
  const int pd = ls.prev_code, nd = ls.code;
  const TensorDesc td = tds[cr.tensor];
  const float eta = ls.eta;
  const uint32_t mode = ls.mode, mask_done = ls.mask_done;
  const uint32_t theta_key = ls.theta_key;
  TA_LOADED("s"(td.param), "s"(td.grad), "s"(td.mom), "s"(td.curv), "s"(td.numel), "s"(td.grad_dtype),
            "s"(td.has_probe), "s"(pd), "s"(nd), "s"(eta), "s"(mode), "s"(mask_done), "s"(theta_key));
  if (skip_epoch == sc.step_id) return;
  const int64_t base = (int64_t)cr.index * kChunk;
  const StepSize ss{-eta, sc.lr, alpha, theta_key};
  if (elem_size(pd) == elem_size(nd)) update_any<ELEM, MOM>(td, pd, nd, base, sc.inv_scale, wd, mu, ss, threadIdx.x, [] { return true; });
  if constexpr (ELEM) return;
  // kSelHist cannot remain after the last scan; never write a mask from a stale range
  if (td.has_probe && !mask_done && mode != kSelHist) {
    mask_chunk(td, base, mode, theta_key, ls.rng_lo, ls.rng_hi, cr.index, cr.tensor, tab->cands, tab->cand_counters);
  }
}

hipError_t launch_update(const DeviceTables& t, const StepScalars& sc, bool elem, bool resize, hipStream_t s) {
  const ResizeGrid rg = resize ? resize_grid(t.plan, 0u, t.n_tensors, t.total_chunks < kResizeBigSet) : ResizeGrid{1u, 0u};
  const bool mom = t.hyper.momentum != 0.0f;
  const auto kernel = elem ? (mom ? k_update<true, true> : k_update<true, false>) : (mom ? k_update<false, true> : k_update<false, false>);
  return launch(kernel, t.total_chunks + rg.grid, kThreads, s, t.dev, t.tensors, t.chunks, t.glob, sc, rg.slots, rg.grid);
}

hipError_t launch_mask_pass(const DeviceTables& t, const StepScalars& sc, hipStream_t s) {
  const uint32_t grid = t.total_chunks < t.persistent_grid ? t.total_chunks : t.persistent_grid;
  return launch(k_mask_pass, grid, kThreads, s, t.dev, t.tensors, t.chunks, t.glob, sc, grid);
}

}  // namespace triaccel
