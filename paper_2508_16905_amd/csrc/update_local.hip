// gfx950 kernels for sets bound by their launches: k_update_local does what the per-layer kernel, the fallback
// histogram pass, the fused update + cast and the first launch of the in-place resize do one after the other on
// larger sets, k_select_tail what the mask pass and the threshold resolution do; with step sizes per element, where the
// update comes last, k_decide_select takes the place of the per-layer kernel, the histogram pass and most of the resolution.
#include "resize_body.h"
#include "select_local.h"

namespace triaccel {

// Arrival counter of a tensor, in a cache line of its own.
__device__ __forceinline__ uint32_t* arrival(uint32_t* arrived, uint32_t l) { return arrived + (size_t)l * kCandCounterStride; }

// Puts back the curvature and the mask words of a chunk.
__device__ __forceinline__ void restore_chunk(const TensorDesc& td, int64_t base, const EmaUndo& undo) {
  const int32_t left = chunk_left(base, td.numel);
  const Tail tail = tail_of(left, threadIdx.x);
  uint32_t h[kRows][4];
  const uint32_t ht = load_chunk<4>(undo.h, left, tail, h);
  void* const hp = chunk_of<4>(static_cast<void*>(td.curv), base);
  const Rows rows = rows_of<4>(hp, left);
#pragma unroll
  for (int r = 0; r < kRows; ++r) store_words<4>(rows, r, threadIdx.x, h[r]);
  if (tail.any) store_tail<kFP32>(hp, tail, ht);
  int64_t word;
  if (mask_word_of(td, base, word)) as_global<uint32_t>(td.mask)[word] = as_global<uint32_t>(undo.mask)[word - (base >> 5)];
}

// Every workgroup of a chunk adds up its tensor's chunk records (at most kLocalMaxChunks x 32 bytes, from
// the caches) and takes the layer's decisions itself, each the same ones, while the chunk's own data is on
// the way.  No workgroup waits for another: what the decisions and the selection read of the layer's record was
// copied aside by the statistics kernel (LayerIn), so that the record may be written while the others
// run.  (An arrival counter per
// tensor instead, with the last workgroup writing, cost one atomic per chunk: with the counters side by side
// in a cache line 20 ns each, 205 us instead of 35 on the ResNet-18 set.)
//
// The first `select_wgs` workgroups settle the thresholds of the tensors whose listed keys suffice (select_local): they
// need nothing of this launch, and they take as long as the streaming around them or less.  In a launch of their own
// afterwards they cost 10 to 13 us of a probed step.  For the other tensors the chunk workgroups also count |h| into the
// tensor's histogram, and the last of the tensor scans it; k_select_tail does what is left of their selection.
//
// Measured, per step: the decisions in here against launches of their own, two-layer perceptron (4 tensors, 0.1 M)
// 13.4 -> 8.8 us, EfficientNet-B0 set 23.4 -> 19.5 (16-bit gradients, no probe) and 65.7 -> 57.1 (probed), ResNet-18 set
// 54.6 -> 50.7 and 102.4 -> 94.5; the selection in here against k_select_tail, with a probe: the perceptron with fp16
// gradients and the result read each time 35.0 -> 29.0, EfficientNet-B0 49.2 -> 39.2, ResNet-18 84.5 -> 73.3, 41 ragged
// tensors of 9.7 M with the Fisher source 59.5 -> 50.0, 4000 tensors of 10 to 300 elements 175 -> 75.
// UNDO: after k_stats_ema, so a probed step that turns out to be skipped puts back what that kernel overwrote.  (As a
// parameter of the launch it cost the probed form twice the scalar registers kept in vector registers, and the ResNet-18
// set 0.4 us a step.)
template <bool MOM, bool PROBED, bool UNDO>
__global__ __launch_bounds__(kThreads) void k_update_local(const StepTables* __restrict__ tab, const TensorDesc* __restrict__ tds,
                                                           const ChunkRef* __restrict__ chunks, GlobalDev* glob, StepScalars arg,
                                                           uint32_t select_wgs) {
  __shared__ LayerShared sh_layer;
  __shared__ union {
    HistShared hist;
    LocalSelectShared select;
  } shared;
  HistShared& sh = shared.hist;
  __shared__ LayerOut s_decision;
  __shared__ uint32_t s_last;
  if constexpr (PROBED) {
    if (blockIdx.x < select_wgs) {
      if (blockIdx.x < tab->n_tensors)
        select_local(blockIdx.x, *tab, tds, glob, step_scalars(arg, *tab), tab->hyper, sh_layer, shared.select);
      return;
    }
  }
  const ChunkRef cr = chunks[blockIdx.x - (PROBED ? select_wgs : 0u)];
  const StepScalars sc = step_scalars(arg, *tab);
  const Hyper hp = tab->hyper;
  const uint64_t skip_epoch = glob->skip_epoch;
  const bool skip = skip_epoch == sc.step_id;
  const StatPartial* const partials = tab->partials;
  const EmaPartial* const ema_partials = tab->ema_partials;
  const TensorDesc td = tds[cr.tensor];
  LayerDev& ls = tab->layers[cr.tensor];
  const LayerIn in = tab->inputs[cr.tensor];
  TA_LOADED("s"(td.param), "s"(td.grad), "s"(td.mom), "s"(td.curv), "s"(td.numel), "s"(td.first_chunk), "s"(td.grad_dtype),
            "s"(td.has_probe), "s"(in.v), "s"(in.lambda), "s"(in.lambda_ctrl), "s"(in.code), "s"(in.prev_code), "s"(in.applied_steps),
            "s"(in.lambda_power), "s"(td.n_chunks), "s"(partials), "s"(ema_partials), "s"(hp.weight_decay), "s"(hp.momentum),
            "s"(hp.beta_var), "s"(hp.tau_low), "s"(hp.tau_high), "s"(hp.tau_curv), "s"(hp.alpha), "s"(hp.ctrl_interval),
            "s"(hp.lambda_source));
  if (skip) {
    if constexpr (UNDO) {
      if (td.has_probe) {
        // the curvature kernel did not know it yet
        const int64_t base = (int64_t)cr.index * kChunk;
        restore_chunk(td, base, ema_undo(tab->undo_h, tab->undo_mask, td, base));
        if (cr.index == 0) reset_cand_counters(tab->cand_counters, cr.tensor);
      }
    }
    if (threadIdx.x == 0 && cr.index == 0) {
      ls.found_inf = (ls.found_epoch == sc.step_id) ? 1u : 0u;
      if (cr.tensor == 0) step_record(glob, tab->host_result, sc, hp, true);
    }
    return;
  }
  const int64_t base = (int64_t)cr.index * kChunk;
  const bool probed = PROBED && td.has_probe != 0;
  const LayerAcc acc = layer_accumulate<PROBED>(td, partials, ema_partials, probed);
  // The chunk's own loads are under way while the sums are reduced and the decisions taken (2-3 % of a step from
  // 11 M to 30 M parameters against loading after them).  They are of no use if the layer changes its storage size
  // (50 M parameters all changing: 312 us a step with them, 238 without); a layer that did so at its last step, or has
  // its first, is taken to be about to do it.
  const bool early = in.applied_steps != 0 && elem_size(in.code) == elem_size(in.prev_code);
  const int pd = in.code;
  int nd;
  StepSize ss;
  const auto decide = [&]() {
    const LayerSums sums = layer_reduce<PROBED>(acc, td.numel, sh_layer);
    const LayerOut o = layer_decide(in, sums, probed, sc.lr, hp);
    if (threadIdx.x == 0) s_decision = o;  // for this thread alone, below
    nd = (int)uniform((uint32_t)o.code);
    ss = StepSize{-u2f(uniform(f2u(o.eta))), sc.lr, hp.alpha, 0u};
    return elem_size(pd) == elem_size(nd);
  };
  bool in_place = early || decide();
  if (in_place)
    in_place = update_any<false, MOM>(td, pd, nd, base, sc.inv_scale, hp.weight_decay, hp.momentum, ss, threadIdx.x,
                                      [&]() { return early ? decide() : true; });
  // launch 0 of the in-place resize: slot r of the tensor is the workgroup of its chunk r
  if (!in_place) resize_item<false, MOM>(td, pd, nd, ss, *tab, 0u, cr.index, sc);
  // read again from shared memory: kept, they went to memory and back for want of registers
  EmaTotals ema{0, 0, 0, 0, 0};
  if constexpr (PROBED) ema = layer_ema(sh_layer);
  uint32_t k = 0;
  int outcome = kOutListed;
  if constexpr (PROBED) {
    if (probed) {
      const SelNow now = in.plan;
      k = topk_count(td.numel, hp.sparsity_ppm, hp.topk_abs);
      outcome = select_outcome(td, now, ema, k);
      if (outcome == kOutHist) {
        const Window w = first_window(now, ema.maxkey);
        for (int b = threadIdx.x; b < kHistBins; b += kThreads) sh.hist[b] = 0;
        __syncthreads();
        uint32_t above = 0;
        hist_chunk(td, base, w, sh.hist, now.predicted != 0, above);
        flush_hist(sh.hist, w.bins, tab->hist + (size_t)cr.tensor * kHistBins);
        above = wave_sum(above);
        if ((threadIdx.x & (kWave - 1)) == 0 && above) atomicAdd(&ls.acc_above, above);
        // This workgroup's counts (device-scope atomics) are complete before its arrival is counted.  With a
        // release fence instead the first probed step of the ResNet-18 set took 833 us, 163 without.
        published_before_here();
        __syncthreads();
      }
    }
  }
  if (threadIdx.x == 0 && cr.index == 0) {
    // (kOutListed: select_local; kOutHist: below)
    if (probed && outcome == kOutFewNonzero) select_setup(td, ls, glob, in.plan, ema, k, outcome, sc.step_id);
    layer_publish(cr.tensor, ls, s_decision, glob, tab->trans_list, tab->n_tensors, sc.step_id);
    if (cr.tensor == 0) step_record(glob, tab->host_result, sc, hp, false);
  }
  if constexpr (PROBED) {
    if (cr.index == 0 && outcome != kOutListed) reset_cand_counters(tab->cand_counters, cr.tensor);  // drop what was listed
    if (outcome != kOutHist) return;
    if (threadIdx.x == 0) {
      const bool last = atomicAdd(arrival(tab->arrived, cr.tensor), 1u) + 1u == td.n_chunks;
      if (last) {
        *arrival(tab->arrived, cr.tensor) = 0;
        select_setup(td, ls, glob, in.plan, ema, k, outcome, sc.step_id);
      }
      s_last = last ? 1u : 0u;
    }
    __syncthreads();
    if (!s_last) return;
    // the scan reads what the other workgroups added with device-scope loads
    select_scan(cr.tensor, td, ls, glob, tab->hist, sc.step_id, sh.hist, sh.part, sh.out, true);
    select_serial(cr.tensor, td, ls, glob, tab->hist, sc.step_id, sh.hist, sh.part, sh.out, 8);
  }
}

// Before the element-wise form of the update on sets of that size: what k_update_local does on probed steps, less the update,
// which needs the thresholds.  Workgroups [0, select_wgs) settle the thresholds of the tensors whose keys suffice
// (select_local), one each; [select_wgs, 2 select_wgs) take the layers' decisions; the others make the fallback histogram
// pass, each over a run of chunks, and leave at once if no tensor of the run needs it.  They take the outcome of a
// tensor from the chunks' records themselves, so that none waits for another.  With a kernel each for the decisions, for the
// histograms and for the thresholds the steady state took two launches more; figures at kDecideMaxChunks.  Bound by latency: 6
// to 10 us up to 16 M elements.
// UNDO: after k_stats_ema; on a skipped step the last kind puts back what that kernel overwrote.
template <bool UNDO>
__global__ __launch_bounds__(kThreads) void k_decide_select(const StepTables* __restrict__ tab, const TensorDesc* __restrict__ tds,
                                                            const ChunkRef* __restrict__ chunks, GlobalDev* glob, StepScalars arg,
                                                            uint32_t select_wgs, uint32_t hist_wgs) {
  __shared__ LayerShared sh_layer;
  __shared__ union {
    HistShared hist;
    LocalSelectShared select;
  } shared;
  __shared__ uint32_t s_last;
  const StepScalars sc = step_scalars(arg, *tab);
  const uint32_t n_tensors = tab->n_tensors;
  if (blockIdx.x < select_wgs) {
    if (blockIdx.x < n_tensors) select_local(blockIdx.x, *tab, tds, glob, sc, tab->hyper, sh_layer, shared.select);
    return;
  }
  const Hyper hp = tab->hyper;
  const uint64_t skip_epoch = glob->skip_epoch;
  const bool skip = skip_epoch == sc.step_id;
  LayerDev* const layers = tab->layers;
  const LayerIn* const inputs = tab->inputs;
  const EmaPartial* const ema_partials = tab->ema_partials;
  if (blockIdx.x < 2 * select_wgs) {
    const uint32_t l = blockIdx.x - select_wgs;
    if (l >= n_tensors) return;
    const TensorDesc td = tds[l];
    LayerDev& ls = layers[l];
    const LayerIn in = inputs[l];
    if (skip) {
      if (UNDO && td.has_probe) reset_cand_counters(tab->cand_counters, l);
      if (threadIdx.x == 0) {
        ls.found_inf = (ls.found_epoch == sc.step_id) ? 1u : 0u;
        if (l == 0) step_record(glob, tab->host_result, sc, hp, true);
      }
      return;
    }
    const bool probed = td.has_probe != 0;
    const LayerSums sums = layer_reduce<true>(layer_accumulate<true>(td, tab->partials, ema_partials, probed), td.numel, sh_layer);
    const uint32_t k = topk_count(td.numel, hp.sparsity_ppm, hp.topk_abs);
    const int outcome = probed ? select_outcome(td, in.plan, sums.ema, k) : (int)kOutListed;
    if (outcome != kOutListed) reset_cand_counters(tab->cand_counters, l);  // drop what was listed
    if (threadIdx.x != 0) return;
    // (kOutListed: select_local; kOutHist: below)
    if (outcome == kOutFewNonzero) select_setup(td, ls, glob, in.plan, sums.ema, k, outcome, sc.step_id);
    layer_publish(l, ls, layer_decide(in, sums, probed, sc.lr, hp), glob, tab->trans_list, n_tensors, sc.step_id);
    if (l == 0) step_record(glob, tab->host_result, sc, hp, false);
    return;
  }
  const uint32_t total_chunks = tab->total_chunks, part = blockIdx.x - 2 * select_wgs;
  const uint32_t per = (total_chunks + hist_wgs - 1) / hist_wgs;
  const uint32_t c1 = min((part + 1) * per, total_chunks);
  uint32_t c = min(part * per, total_chunks);
  HistShared& sh = shared.hist;
  while (c < c1) {
    const uint32_t l = uniform(chunks[c].tensor);
    const TensorDesc td = tds[l];
    const uint32_t end = min(td.first_chunk + td.n_chunks, c1);
    const uint32_t first = c, mine = end - c;
    c = end;
    if (!td.has_probe) continue;
    if (skip) {
      if constexpr (UNDO)
        for (uint32_t q = first; q < end; ++q) {
          const int64_t base = (int64_t)(q - td.first_chunk) * kChunk;
          restore_chunk(td, base, ema_undo(tab->undo_h, tab->undo_mask, td, base));
        }
      continue;
    }
    if (td.list_all) continue;
    const SelNow now = inputs[l].plan;
    const EmaTotals e = ema_totals(td, ema_partials, sh_layer);
    const uint32_t k = topk_count(td.numel, hp.sparsity_ppm, hp.topk_abs);
    const int outcome = select_outcome(td, now, e, k);
    __syncthreads();  // the sums' shared memory may be written again
    if (outcome != kOutHist) continue;
    LayerDev& ls = layers[l];
    const Window w = first_window(now, e.maxkey);
    for (int b = threadIdx.x; b < kHistBins; b += kThreads) sh.hist[b] = 0;
    __syncthreads();
    uint32_t above = 0;
    for (uint32_t q = first; q < end; ++q) hist_chunk(td, (int64_t)(q - td.first_chunk) * kChunk, w, sh.hist, now.predicted != 0, above);
    flush_hist(sh.hist, w.bins, tab->hist + (size_t)l * kHistBins);
    above = wave_sum(above);
    if ((threadIdx.x & (kWave - 1)) == 0 && above) atomicAdd(&ls.acc_above, above);
    published_before_here();  // as in k_update_local
    __syncthreads();
    if (threadIdx.x == 0) {
      const bool last = atomicAdd(arrival(tab->arrived, l), mine) + mine == td.n_chunks;
      if (last) {
        *arrival(tab->arrived, l) = 0;
        select_setup(td, ls, glob, now, e, k, outcome, sc.step_id);
      }
      s_last = last ? 1u : 0u;
    }
    __syncthreads();
    if (s_last) {
      select_scan(l, td, ls, glob, tab->hist, sc.step_id, sh.hist, sh.part, sh.out, true);
      select_serial(l, td, ls, glob, tab->hist, sc.step_id, sh.hist, sh.part, sh.out, 8);
    }
    __syncthreads();
  }
}

hipError_t launch_decide_select(const DeviceTables& t, const StepScalars& sc, bool undo, hipStream_t s) {
  const uint32_t select_wgs = (t.n_tensors + 7u) & ~7u;
  // four for a compute unit, which is as fast as eight (the pass is bound by the LDS's atomic adds), or a chunk each; none if
  // there is nothing to count and nothing to put back
  const uint32_t cap = t.persistent_grid / 2;
  const uint32_t hist_wgs = t.all_small && !undo ? 0u : t.total_chunks < cap ? t.total_chunks : cap;
  return launch(undo ? k_decide_select<true> : k_decide_select<false>, 2 * select_wgs + hist_wgs, kThreads, s, t.dev, t.tensors, t.chunks,
                t.glob, sc, select_wgs, hist_wgs);
}

hipError_t launch_update_local(const DeviceTables& t, const StepScalars& sc, bool any_probe, bool undo, hipStream_t s) {
  const bool mom = t.hyper.momentum != 0.0f;
  const auto kernel = !any_probe ? (mom ? k_update_local<true, false, false> : k_update_local<false, false, false>)
                      : undo     ? (mom ? k_update_local<true, true, true> : k_update_local<false, true, true>)
                                 : (mom ? k_update_local<true, true, false> : k_update_local<false, true, false>);
  // a multiple of eight: a chunk's workgroup goes to the same die in every kernel
  const uint32_t select_wgs = any_probe ? (t.n_tensors + 7u) & ~7u : 0u;
  return launch(kernel, select_wgs + t.total_chunks, kThreads, s, t.dev, t.tensors, t.wg_chunks, t.glob, sc, select_wgs);
}

// What is left of the selection after k_update_local or k_decide_select, and before the element-wise form of the update on
// sets of fewer than kLaunchBoundChunks with longer tensors (one launch for the mask pass and the threshold resolution).
// Workgroup l < n_tensors settles tensor l if its listed keys suffice (`local`: if select_local left them).  The `mask_wgs` workgroups after
// those make the mask pass of the other tensors, four chunks at a
// time, and the last workgroup to finish a part of such a tensor settles it among the keys the pass listed; the
// rest take launch 1 of the in-place resize, four chunks of a level at a time.  After k_update_local all of them leave
// at once in the steady state, which costs a step 1.5 us.
template <bool MOM>
__global__ __launch_bounds__(kFinishThreads) void k_select_tail(const StepTables* __restrict__ tab, const TensorDesc* __restrict__ tds,
                                                                GlobalDev* glob, StepScalars arg, uint32_t mask_wgs,
                                                                uint32_t resize_wgs, uint32_t resize_slots, int local) {
  __shared__ SelectShared<kFinishThreads> sh;
  __shared__ uint32_t s_last;
  const StepScalars sc = step_scalars(arg, *tab);
  const uint32_t n_tensors = tab->n_tensors, total_chunks = tab->total_chunks;
  LayerDev* const layers = tab->layers;
  uint32_t* const counters = tab->cand_counters;
  const float beta_h = tab->hyper.beta_curv;
  const uint64_t skip_epoch = glob->skip_epoch;
  const uint32_t pending = glob->mask_pending[sc.step_id & 1u];
  if (blockIdx.x < n_tensors) {
    if (local) {
      TA_LOADED("s"(skip_epoch), "s"(pending));
      if (pending == 0 || skip_epoch == sc.step_id) return;
      // (a step with nothing pending was not a late one, so there is nothing to take back when all leave above)
      if (blockIdx.x == 0 && threadIdx.x == 0)
        glob->select_late = glob->late_epoch == sc.step_id &&
                            (tab->hyper.elementwise == 1 ? n_tensors <= kLateTensors : total_chunks <= kLateChunks);
    }
    const uint32_t l = blockIdx.x;
    const uint32_t listed = threadIdx.x <= kCandLists ? *cand_counter(counters, l, threadIdx.x) : 0u;
    const TensorDesc td = tds[l];
    LayerDev& ls = layers[l];
    // sel_outcome is not written here: it tells the two kinds apart while the records are rewritten
    const uint32_t sel_outcome = ls.sel_outcome;
    const FinishIn in = finish_in(ls);
    TA_LOADED("s"(td.mask), "s"(td.has_probe), "s"(td.cand_cap), "s"(sel_outcome), "s"(in.mode), "s"(in.probes_seen),
              "s"(in.var_hold));
    // (a tensor that select_local settled is no longer in this mode)
    if (skip_epoch == sc.step_id || !td.has_probe || sel_outcome > 1u || in.mode != kSelCand) return;
    select_finish<kFinishThreads, kFinishRegs>(l, td, ls, in, listed, tab->cands, counters, beta_h, sh);
    return;
  }
  if (blockIdx.x >= n_tensors + mask_wgs) {
    const uint32_t count = glob->trans_count[sc.step_id & 1u];
    TA_LOADED("s"(skip_epoch), "s"(count));
    if (count == 0 || skip_epoch == sc.step_id) return;
    resize_items<false, MOM, kFinishThreads / kThreads>(*tab, tds, count, 1u, resize_slots,
                                                        blockIdx.x - n_tensors - mask_wgs, resize_wgs, sc);
    return;
  }
  TA_LOADED("s"(skip_epoch), "s"(pending));
  if (pending == 0 || skip_epoch == sc.step_id) return;
  const uint32_t part = blockIdx.x - n_tensors, parts = mask_wgs;
  const uint32_t per = (total_chunks + parts - 1) / parts;
  const uint32_t c1 = min((part + 1) * per, total_chunks);
  const uint32_t group = uniform(threadIdx.x / kThreads);
  uint32_t c = min(part * per, total_chunks);
  while (c < c1) {
    const uint32_t l = tab->chunks[c].tensor;
    const TensorDesc td = tds[l];
    const uint32_t end = min(td.first_chunk + td.n_chunks, c1);
    const uint32_t mine = end - c;
    LayerDev& ls = layers[l];
    const uint32_t mode = ls.mode;
    if (!td.has_probe || ls.sel_outcome <= 1u || mode == kSelHist) {
      c = end;
      continue;
    }
    const uint32_t theta = ls.theta_key, rng_lo = ls.rng_lo, rng_hi = ls.rng_hi;
    for (uint32_t q = c + group; q < end; q += kFinishThreads / kThreads) {
      const uint32_t index = q - td.first_chunk;
      const int64_t base = (int64_t)index * kChunk;
      mask_chunk<true>(td, base, mode, theta, rng_lo, rng_hi, index, l, tab->cands, counters);
    }
    c = end;
    published_before_here();  // mask words and listed keys are complete before the arrival is counted
    __syncthreads();
    if (threadIdx.x == 0) {
      const bool last = atomicAdd(arrival(tab->arrived, l), mine) + mine == td.n_chunks;
      if (last) *arrival(tab->arrived, l) = 0;
      s_last = last ? 1u : 0u;
    }
    __syncthreads();
    const bool last = s_last != 0;
    __syncthreads();
    if (last) {
      // the resolution reads what the other workgroups listed: nothing older of it in this unit's caches
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      uint32_t listed = 0;
      if (threadIdx.x <= kCandLists)
        listed = __hip_atomic_load(cand_counter(counters, l, threadIdx.x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      select_finish<kFinishThreads, kFinishRegs>(l, td, ls, finish_in(ls), listed, tab->cands, counters, beta_h, sh);
      __syncthreads();
    }
  }
}

static_assert((kResizeTopSmall << 6) >= kLocalMaxChunks && kLaunchBoundChunks <= kResizeBigSet,
              "one subtree stage: the resize of a set of the local form has two launches at most");
hipError_t launch_select_tail(const DeviceTables& t, const StepScalars& sc, bool local, bool resize, hipStream_t s) {
  constexpr uint32_t kGroups = kFinishThreads / kThreads;
  const uint32_t all = (t.total_chunks + kGroups - 1) / kGroups, cap = t.persistent_grid / 8;  // one per CU
  const uint32_t mask_wgs = all < cap ? all : cap;
  ResizeGrid rg{1u, 0u};
  if (resize && t.plan.n_stages > 1) {
    rg = resize_grid(t.plan, 1u, t.n_tensors, true);
    if (rg.grid > cap) rg.grid = cap;
  }
  const auto kernel = t.hyper.momentum != 0.0f ? k_select_tail<true> : k_select_tail<false>;
  return launch(kernel, t.n_tensors + mask_wgs + rg.grid, kFinishThreads, s, t.dev, t.tensors, t.glob, sc, mask_wgs, rg.grid,
                rg.slots, local ? 1 : 0);
}

}  // namespace triaccel
