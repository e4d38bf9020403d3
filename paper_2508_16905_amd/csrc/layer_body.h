// Per-layer assignment (Sec. 3.1, 3.2): the sums over a tensor's chunk records and the decisions taken from
// them, shared by the kernel with one workgroup per tensor and by the update of small sets, in which every
// workgroup takes its layer's decisions itself.
#pragma once
#include "select_body.h"

namespace triaccel {

// Shared memory of layer_sums.
struct LayerShared {
  double s1[kThreads / kWave], s2[kThreads / kWave];
  uint32_t red[5][kThreads / kWave];
};

struct LayerSums {
  double mean, var;  // of the unscaled gradient (population variance)
  EmaTotals ema;
};

// Adds up the records of a tensor's chunks (layer_accumulate, then layer_reduce over the workgroup); all
// kThreads threads call it, the result is the same in all.
// Moments: with every chunk's (n_i, mean_i, M2_i) and the shift K = mean of chunk 0,
//   S1 = sum n_i (mean_i - K),  S2 = sum M2_i + n_i (mean_i - K)^2,
//   mean = K + S1 / n,  M2 = S2 - S1^2 / n     (fp64; fixed order over threads, lanes and wavefronts)
// -- four operations per record and one division in all, where merging records pairwise takes a division
// per pair.  K is one of the means, so S2 is at most about M2 times the number of chunks (chunk 0 far off all the
// others), and the cancellation can multiply the sums' rounding error, some 1e-15, by that factor: below 1e-9 for the
// largest tensor (2^19 chunks), where the variance is kept to 6e-8 (fp32).  Replayed for 400 chunks: ordinary data
// 1e-16 to 1e-15 (pairwise 1e-16), chunk 0 off by 1000 standard deviations 2e-14 to 7e-13.
struct LayerAcc {  // one thread's part
  double shift, s1, s2;
  EmaTotals ema;
};
// PROBED: the step has probed tensors, so there are curvature records; `probed`: this tensor is one of them
// (the records of the others are old ones and are dropped after the loop, which has no branch in it, so that
// the loads of its iterations are all under way together).
template <bool PROBED>
__device__ __forceinline__ LayerAcc layer_accumulate(const TensorDesc& td, const StatPartial* __restrict__ partials,
                                                     const EmaPartial* __restrict__ ema_partials, bool probed) {
  const uint32_t nc = td.n_chunks;
  const StatPartial* const p = partials + td.first_chunk;
  const EmaPartial* const q = ema_partials + td.first_chunk;
  LayerAcc a{p[0].mean, 0.0, 0.0, {0, 0, 0, 0, 0}};
  const double tail = (double)(td.numel - (int64_t)(nc - 1) * kChunk);
#pragma unroll 4
  for (uint32_t c = threadIdx.x; c < nc; c += kThreads) {
    const StatPartial r = p[c];
    EmaPartial x{0, 0, 0, 0};
    if constexpr (PROBED) x = q[c];
    const double n = c + 1 < nc ? (double)kChunk : tail;
    const double d = r.mean - a.shift;
    const double nd = n * d;
    a.s1 += nd;
    a.s2 += fma(nd, d, r.m2);
    if constexpr (PROBED) {
      a.ema.above += x.above_zeros & 0xffffu;
      a.ema.zeros += x.above_zeros >> 16;
      a.ema.maxkey = max(a.ema.maxkey, x.maxkey);
      a.ema.listed += x.listed;
      a.ema.nonfin |= x.nonfinite;
    }
  }
  if (!probed) a.ema = EmaTotals{0, 0, 0, 0, 0};
  return a;
}

// The curvature totals of the wavefronts' sums that layer_reduce left in shared memory (after its barrier).
__device__ __forceinline__ EmaTotals layer_ema(const LayerShared& sh) {
  EmaTotals e{0, 0, 0, 0, 0};
#pragma unroll
  for (int w = 0; w < kThreads / kWave; ++w) {
    e.above += sh.red[0][w];
    e.zeros += sh.red[1][w];
    e.maxkey = max(e.maxkey, sh.red[2][w]);
    e.listed += sh.red[3][w];
    e.nonfin |= sh.red[4][w];
  }
  return EmaTotals{uniform(e.above), uniform(e.zeros), uniform(e.maxkey), uniform(e.listed), uniform(e.nonfin)};
}

template <bool PROBED>
__device__ __forceinline__ LayerSums layer_reduce(const LayerAcc& a, int64_t numel, LayerShared& sh) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  double s1 = wave_sum_f64(a.s1);
  double s2 = wave_sum_f64(a.s2);
  EmaTotals e = a.ema;
  if constexpr (PROBED) {
    e.above = wave_sum(e.above);
    e.zeros = wave_sum(e.zeros);
    e.maxkey = wave_max(e.maxkey);
    e.listed = wave_sum(e.listed);
    e.nonfin = wave_or(e.nonfin);
  }
  if (lane == 0) {
    sh.s1[wave] = s1;
    sh.s2[wave] = s2;
    if constexpr (PROBED) {
      sh.red[0][wave] = e.above;
      sh.red[1][wave] = e.zeros;
      sh.red[2][wave] = e.maxkey;
      sh.red[3][wave] = e.listed;
      sh.red[4][wave] = e.nonfin;
    }
  }
  __syncthreads();
  s1 = s2 = 0.0;
#pragma unroll
  for (int w = 0; w < kThreads / kWave; ++w) {
    s1 += sh.s1[w];
    s2 += sh.s2[w];
  }
  if constexpr (PROBED) e = layer_ema(sh);
  else e = EmaTotals{0, 0, 0, 0, 0};
  const double n = (double)numel;
  const double m2 = s2 - s1 * s1 / n;
  // only a negative rounding error is cut off: an unscaled gradient that overflowed leaves NaN here, and the
  // precision rule's comparisons then choose FP32
  return LayerSums{a.shift + s1 / n, (m2 < 0.0 ? 0.0 : m2) / n, e};
}

__device__ __forceinline__ LayerIn layer_in(const LayerDev& ls) {
  return LayerIn{ls.v, ls.lambda, ls.lambda_ctrl, ls.lambda_power, ls.code, ls.prev_code, ls.applied_steps, 0u, select_plan(ls)};
}
struct LayerOut {
  float mean, var, v, lambda, lambda_ctrl, eta;
  int32_t code, prev;
  uint32_t applied_steps, curv_nonfinite;
};

// Variance EMA (Sec. 3.1 first equation), precision rule (second equation) with curvature promotion
// (Sec. 3.2), step size eta_l (Sec. 3.2).
__device__ __forceinline__ LayerOut layer_decide(const LayerIn& in, const LayerSums& s, bool probed, float lr,
                                                 const Hyper& hp) {
  LayerOut o;
  o.applied_steps = in.applied_steps + 1;
  o.mean = (float)s.mean;
  o.var = (float)s.var;
  o.v = o.applied_steps == 1 ? (float)s.var
                             : (float)((double)hp.beta_var * (double)in.v + (1.0 - (double)hp.beta_var) * s.var);
  // lambda_l = largest |h_i| (always inside the mask)
  o.lambda = probed ? u2f(s.ema.maxkey) : in.lambda;
  o.curv_nonfinite = probed ? s.ema.nonfin : 0u;
  if (hp.lambda_source == 1) o.lambda = in.lambda_power;
  o.prev = o.code = in.code;
  o.lambda_ctrl = in.lambda_ctrl;
  if (o.applied_steps % (uint32_t)hp.ctrl_interval == 0) {
    o.lambda_ctrl = o.lambda;
    o.code = (o.v < hp.tau_low) ? kFP16 : (o.v < hp.tau_high) ? kBF16 : kFP32;
    if (o.lambda_ctrl > hp.tau_curv && o.code < kFP32) o.code += 1;
  }
  const float den = fmaf(hp.alpha, o.lambda_ctrl, 1.0f);
  o.eta = lr / den;
  return o;
}

// Writes the layer's record after an applied step (one thread); a layer whose storage size changes joins
// the step's list.
__device__ __forceinline__ void layer_publish(uint32_t l, LayerDev& ls, const LayerOut& o, GlobalDev* glob,
                                              uint32_t* trans_list, uint32_t n_tensors, uint64_t step_id) {
  ls.found_inf = 0;
  ls.applied_steps = o.applied_steps;
  ls.mean = o.mean;
  ls.var = o.var;
  ls.v = o.v;
  ls.lambda = o.lambda;
  ls.lambda_ctrl = o.lambda_ctrl;
  ls.curv_nonfinite = o.curv_nonfinite;
  ls.prev_code = o.prev;
  ls.code = o.code;
  ls.eta = o.eta;
  if (elem_size(o.code) != elem_size(o.prev)) {
    const uint32_t slot = atomicAdd(&glob->trans_count[step_id & 1u], 1u);
    trans_list[(step_id & 1u) * n_tensors + slot] = l;
  }
}

// The step's global record (one thread of one workgroup): loss-scale schedule, result for the host, the
// other parity's counters.
__device__ __forceinline__ void step_record(GlobalDev* glob, GlobalDev* host_result, const StepScalars& sc, const Hyper& hp,
                                            bool skip) {
  glob->trans_count[(sc.step_id + 1u) & 1u] = 0;
  glob->hist_pending[(sc.step_id + 1u) & 1u] = 0;
  glob->mask_pending[(sc.step_id + 1u) & 1u] = 0;
  float next = sc.loss_scale;
  if (skip) {
    glob->good_steps = 0;
    next = sc.loss_scale * hp.scale_backoff;
  } else {
    const int32_t good = glob->good_steps + 1;
    if (good >= hp.growth_interval) {
      glob->good_steps = 0;
      next = sc.loss_scale * hp.scale_growth;
    } else {
      glob->good_steps = good;
    }
  }
  glob->res_skipped = skip ? 1 : 0;
  glob->res_next_scale = next;
  glob->res_step_id = sc.step_id;
  // the host's copy, written straight into pinned host memory (read after the stream has been
  // waited for): no separate device-to-host copy in the stream
  host_result->res_skipped = skip ? 1 : 0;
  host_result->res_next_scale = next;
  host_result->res_step_id = sc.step_id;
}

}  // namespace triaccel
