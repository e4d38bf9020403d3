// Exact top-k threshold selection: device functions shared by the kernels that carry its parts.
#pragma once
#include "device_util.h"

namespace triaccel {

// ---------------------------------------------------------------------------------------------
// Threshold selection (exact k-th largest |h_i| per tensor) on the 31-bit magnitude keys,
// organised so that a probed step normally needs NO pass over h beyond the one that creates it:
//
//   * From the thresholds of the last probed steps (up to three) the library predicts this
//     step's threshold and a BAND around it (a few times the error the last predictions made).
//   * The EMA kernel writes a provisional mask (bit = key at or above the band), lists the keys
//     inside the band, and counts the keys above it.
//   * If the k-th largest key falls inside the band (count above < k <= count above + listed),
//     the listed keys resolve theta exactly and only their mask bits are patched.
//   * Otherwise (no prediction yet, prediction off, too many keys to list) the tensor falls
//     back to a radix select by histogram passes over h and a separate mask pass.
//   * Tensors with at most kListAllMax elements list all their non-zero keys and select from the list; in sets bound by
//     their launches the keys are not listed but read from h (select_local).
// ---------------------------------------------------------------------------------------------
struct Window {
  uint32_t lo, shift, bins;
  uint32_t hi;  // keys in [lo, hi) are counted; hi <= lo + (bins << shift)
};

// Flush a workgroup's LDS histogram to the tensor's global one and clear it.
__device__ __forceinline__ void flush_hist(uint32_t* s_hist, uint32_t bins, uint32_t* g_hist) {
  __syncthreads();
  for (uint32_t b = threadIdx.x; b < bins; b += kThreads) {
    const uint32_t v = s_hist[b];
    if (v) {
      atomicAdd(&g_hist[b], v);
      s_hist[b] = 0;
    }
  }
  __syncthreads();
}

__device__ __forceinline__ void hist_chunk(const TensorDesc& td, int64_t base, const Window& w, uint32_t* s_hist,
                                           bool count_above, uint32_t& above) {
  uint32_t h[kRows][4];
  const int32_t left = chunk_left(base, td.numel);
  const Tail tail = tail_of(left, threadIdx.x);
  const uint32_t ht = load_chunk<4>(chunk_of<4>(td.curv, base), left, tail, h);
  const auto count = [&](uint32_t bits) {
    const uint32_t key = bits & 0x7fffffffu;  // what lies past the end reads as 0 and is never counted
    if (key != 0u && key >= w.lo) {
      if (key < w.hi) atomicAdd(&s_hist[(key - w.lo) >> w.shift], 1u);
      else if (count_above) ++above;
    }
  };
#pragma unroll
  for (int r = 0; r < kRows; ++r)
#pragma unroll
    for (int i = 0; i < 4; ++i) count(h[r][i]);
  if (tail.any) count(ht);
}

// ---------------------------------------------------------------------------------------------
// Rank search in an LDS histogram: find the bin, counted from the top, that holds the r-th
// largest key (1 <= r <= total).  All NT threads of the workgroup call it; results are broadcast.
// ---------------------------------------------------------------------------------------------
struct BinHit {
  uint32_t bin;     // bin holding the r-th largest key
  uint32_t higher;  // number of keys in bins above it
  uint32_t count;   // keys in that bin
};
template <int NT>
__device__ __forceinline__ BinHit find_rank_from_top(const uint32_t* s_hist, uint32_t bins, uint32_t r, uint32_t* s_part,
                                                     uint32_t* s_out) {
  // Every thread sums its run of bins and every wavefront its threads; each wavefront walks the wavefront sums
  // from the top, and the one that holds the rank finds the lane in a scan and the bin in the lane's run.  Two
  // barriers and no serial walk longer than a run (2 bins of 2048 with 1024 threads).
  constexpr int PER = kHistBins / NT, NW = NT / kWave;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const uint32_t b0 = threadIdx.x * PER;
  uint32_t v[PER], sum = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    v[i] = b0 + i < bins ? s_hist[b0 + i] : 0u;
    sum += v[i];
  }
  const uint32_t incl = wave_scan(sum), total = last_lane(incl);
  if (lane == 0) s_part[wave] = total;
  __syncthreads();
  uint32_t higher = 0;  // keys in wavefronts above the one that holds the rank
  int hit = NW - 1;
  for (; hit > 0; --hit) {
    const uint32_t p = s_part[hit];
    if (higher + p >= r) break;
    higher += p;
  }
  if (wave == hit) {
    const uint32_t from_here = total - incl + sum;  // sum over lanes >= this one
    const unsigned long long reach = __ballot(higher + from_here >= r);
    const int pick = reach ? 63 - __clzll(reach) : 0;  // the highest lane from which the top reaches rank r
    if (lane == pick) {
      uint32_t acc = higher + from_here - sum;
      uint32_t bin = b0, cnt = v[0];
#pragma unroll
      for (int i = PER - 1; i > 0; --i) {
        if (acc + v[i] >= r) {
          bin = b0 + i;
          cnt = v[i];
          break;
        }
        acc += v[i];
      }
      s_out[0] = bin;
      s_out[1] = acc;
      s_out[2] = cnt;
    }
  }
  __syncthreads();
  return BinHit{s_out[0], s_out[1], s_out[2]};
}

__device__ __forceinline__ uint32_t topk_count(int64_t n, uint32_t s_ppm, uint32_t k_abs) {
  // a fixed k if given, else k = n - floor(n * s / 1e6); clamped to [1, n]; n < 2^31 so the
  // product fits 64 bits
  int64_t k = k_abs ? (int64_t)k_abs : n - (int64_t)(((uint64_t)n * (uint64_t)s_ppm) / 1000000ull);
  if (k < 1) k = 1;
  if (k > n) k = n;
  return (uint32_t)k;
}

// ---------------------------------------------------------------------------------------------
// After the EMA pass: what the sums of its per-chunk records say about the threshold.
// ---------------------------------------------------------------------------------------------
struct EmaTotals {
  uint32_t above, zeros, maxkey, listed, nonfin;
};

__device__ __forceinline__ SelNow select_plan(const LayerDev& ls) {
  return SelNow{ls.use_band, ls.band_lo, ls.band_hi, ls.predicted, ls.win_lo, ls.win_hi, ls.win_shift, ls.win_bins};
}

enum SelOutcome : int {
  kOutListed = 0,     // the listed keys settle the threshold (band hit, or small tensor)
  kOutFewNonzero = 1, // fewer non-zero keys than k: theta = 0
  kOutHist = 2,       // histogram passes
};
__device__ __forceinline__ int select_outcome(const TensorDesc& td, const SelNow& now, const EmaTotals& e, uint32_t k) {
  if (td.list_all) return kOutListed;
  if (k > (uint32_t)td.numel - e.zeros) return kOutFewNonzero;
  if (now.use_band && e.above < k && k <= e.above + e.listed && e.listed <= td.cand_cap) return kOutListed;
  return kOutHist;
}

// Window of the first histogram pass: the predicted one if there is one; else the two octaves
// below the largest key, where the threshold of a top-k selection normally lies (nothing is above that
// window, so the count above it is known).
__device__ __forceinline__ Window first_window(const SelNow& now, uint32_t maxkey) {
  if (now.predicted) return Window{now.win_lo, now.win_shift, now.win_bins, now.win_hi};
  const uint32_t span = (uint32_t)kHistBins << kFirstShift;
  const uint32_t hi = maxkey + 1u;
  return Window{hi > span ? hi - span : 0u, kFirstShift, (uint32_t)kHistBins, hi};
}

// Lays down the selection state of tensor l for the outcome (one thread).
__device__ __forceinline__ void select_setup(const TensorDesc& td, LayerDev& ls, GlobalDev* glob, const SelNow& now,
                                             const EmaTotals& e, uint32_t k, int outcome, uint64_t step_id) {
  const uint32_t nonzero = (uint32_t)td.numel - e.zeros;
  // diagnostic: 0 small tensor, 1 band held, 2 no band this step, 3 threshold above the band,
  // 4 threshold below the band, 5 too many keys listed, 6 fewer non-zero keys than k
  ls.sel_listed = e.listed;
  ls.sel_outcome = td.list_all ? 0u
                   : k > nonzero ? 6u
                   : !now.use_band ? 2u
                   : e.above >= k ? 3u
                   : k > e.above + e.listed ? 4u
                   : e.listed > td.cand_cap ? 5u : 1u;
  ls.nonzero = nonzero;
  ls.k_rem = k;
  ls.passes = 1;
  ls.acc_maxkey = e.maxkey;
  if (outcome != kOutListed) atomicAdd(&glob->mask_pending[step_id & 1u], 1u);
  if (outcome == kOutListed) {
    ls.mode = kSelCand;
    ls.mask_done = 1;
    if (td.list_all) {
      ls.above = 0;
      ls.rng_lo = 0;
      ls.rng_hi = 0x80000000u;
    } else {
      ls.above = e.above;
      ls.rng_lo = now.band_lo;
      ls.rng_hi = now.band_hi;
      ls.dens_count = e.listed;
      ls.dens_width = now.band_hi - now.band_lo;
    }
  } else if (outcome == kOutFewNonzero) {
    ls.mode = kSelExact;
    ls.mask_done = 0;
    ls.theta_key = 0;
    ls.above = nonzero;
    ls.sel_count = 0;
  } else {
    const Window w = first_window(now, e.maxkey);
    ls.mode = kSelHist;
    ls.mask_done = 0;
    ls.above = 0;
    ls.count_above = now.predicted;
    ls.win_lo = w.lo;
    ls.win_hi = w.hi;
    ls.win_shift = w.shift;
    ls.win_bins = w.bins;
    atomicAdd(&glob->hist_pending[step_id & 1u], 1u);
  }
}

// ---------------------------------------------------------------------------------------------
// Scan after a histogram pass, by one workgroup for one tensor in mode kSelHist: read the
// tensor's histogram (from memory, clearing it, or already complete in LDS), and decide whether
// theta is now exact, lies in a range whose keys can be listed by the mask pass, or needs a finer
// histogram.  Uniform over the workgroup.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ void select_scan(uint32_t l, const TensorDesc& td, LayerDev& ls, GlobalDev* glob, uint32_t* hist,
                            uint64_t step_id, uint32_t* s_hist, uint32_t* s_part, uint32_t* s_out, bool from_global) {
  const uint32_t bins = ls.win_bins, lo = ls.win_lo, shift = ls.win_shift;
  uint32_t* gh = hist + (size_t)l * kHistBins;
  uint32_t local = 0;
  for (uint32_t b = threadIdx.x; b < kHistBins; b += kThreads) {
    uint32_t v;
    if (from_global) {
      // counted by other workgroups of the running kernel: read at device scope
      v = (b < bins) ? __hip_atomic_load(&gh[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
      s_hist[b] = v;
      if (v) gh[b] = 0;
    } else {
      v = (b < bins) ? s_hist[b] : 0u;
    }
    local += v;
  }
  local = wave_sum(local);
  if ((threadIdx.x & (kWave - 1)) == 0) s_part[threadIdx.x / kWave] = local;
  __syncthreads();
  const uint32_t in_window = s_part[0] + s_part[1] + s_part[2] + s_part[3];
  __syncthreads();
  const uint32_t k = ls.k_rem;
  // counted by this pass (same remark), or known
  const uint32_t above = ls.count_above ? __hip_atomic_load(&ls.acc_above, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : ls.above;
  const bool missed = above >= k || above + in_window < k;
  BinHit hit{0, 0, 0};
  if (!missed) hit = find_rank_from_top<kThreads>(s_hist, bins, k - above, s_part, s_out);
  __syncthreads();
  if (threadIdx.x == 0) {
    ls.acc_above = 0;
    ls.count_above = 0;
    ls.hist_arrived = 0;
    ls.passes = ls.passes + 1;
    if (missed) {
      // The window does not contain theta.  Continue with what lies on the side where it must be:
      // between the window and the largest key (nothing is above that), or below the window (then
      // every key counted so far is above the new window).
      const uint32_t old_hi = ls.win_hi;
      uint32_t new_lo, new_hi;
      if (above >= k) {
        new_lo = old_hi;
        new_hi = ls.acc_maxkey + 1u;  // acc_maxkey >= old_hi: some key lies above the window
        ls.above = 0;
      } else {
        new_lo = 0;
        new_hi = lo;
        ls.above = above + in_window;
      }
      uint32_t ns = 0;
      while (ns < kFullShift && ((uint32_t)kHistBins << ns) < new_hi - new_lo) ++ns;
      ls.win_lo = new_lo;
      ls.win_hi = new_hi;
      ls.win_shift = ns;
      ls.win_bins = kHistBins;
      ls.window_missed = 1;
    } else {
      const uint32_t new_lo = lo + (hit.bin << shift);
      // the bin ends where the window ends (its last bin may be cut short)
      const uint32_t new_hi = min(new_lo + (1u << shift), ls.win_hi);
      ls.above = above + hit.higher;
      ls.sel_count = hit.count;
      ls.dens_count = hit.count;
      ls.dens_width = 1u << shift;
      if (shift == 0) {
        ls.mode = kSelExact;
        ls.theta_key = new_lo;
        atomicSub(&glob->hist_pending[step_id & 1u], 1u);
      } else if (hit.count <= td.cand_cap) {
        ls.mode = kSelCand;
        ls.rng_lo = new_lo;
        ls.rng_hi = new_hi;
        atomicSub(&glob->hist_pending[step_id & 1u], 1u);
      } else {
        const uint32_t ns = shift > (uint32_t)kHistBits ? shift - kHistBits : 0u;
        ls.win_lo = new_lo;
        ls.win_hi = new_hi;
        ls.win_shift = ns;
        ls.win_bins = 1u << (shift - ns);
      }
    }
  }
  __syncthreads();
}

// After a scan that was not the last: up to `serial_rounds` further passes over the whole tensor by this
// workgroup alone.
__device__ __forceinline__ void select_serial(uint32_t l, const TensorDesc& td, LayerDev& ls, GlobalDev* glob, uint32_t* hist,
                                              uint64_t step_id, uint32_t* s_hist, uint32_t* s_part, uint32_t* s_out,
                                              int serial_rounds) {
  for (int extra = 0; extra < serial_rounds; ++extra) {
    if (ls.mode != kSelHist) break;  // written before the barrier that ends the scan
    for (int b = threadIdx.x; b < kHistBins; b += kThreads) s_hist[b] = 0;
    __syncthreads();
    // after a scan the number of keys above the window is known
    const Window w2{ls.win_lo, ls.win_shift, ls.win_bins, ls.win_hi};
    uint32_t unused = 0;
    for (uint32_t q = 0; q < td.n_chunks; ++q) {
      const int64_t b2 = (int64_t)q * kChunk;
      hist_chunk(td, b2, w2, s_hist, false, unused);
    }
    __syncthreads();
    select_scan(l, td, ls, glob, hist, step_id, s_hist, s_part, s_out, false);
  }
}

// ---------------------------------------------------------------------------------------------
// Finish: one workgroup resolves theta among the listed keys (radix select in LDS),
// sets their mask bits, publishes theta / nnz and plans the next probed step: the band and the
// fallback window are centred on the predicted threshold; their widths follow the error the
// recent predictions made.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t abs_diff(uint32_t a, uint32_t b) { return a > b ? a - b : b - a; }

// The fields of a layer's record that the finish reads: loaded together and ahead of the listed keys, instead of
// one after the other where they are used.
struct FinishIn {
  uint32_t mode, above, rng_lo, rng_hi, theta_key, sel_count, nonzero, k_rem, passes, mask_done, probes_seen;
  uint32_t theta_key_last, theta_key_last2, n_theta, pred_ext_key, window_missed, dens_count, dens_width;
  float var_hold, var_ext;
};
__device__ __forceinline__ FinishIn finish_in(const LayerDev& ls) {
  return FinishIn{ls.mode, ls.above, ls.rng_lo, ls.rng_hi, ls.theta_key, ls.sel_count, ls.nonzero, ls.k_rem, ls.passes,
                  ls.mask_done, ls.probes_seen, ls.theta_key_last, ls.theta_key_last2, ls.n_theta, ls.pred_ext_key,
                  ls.window_missed, ls.dens_count, ls.dens_width, ls.var_hold, ls.var_ext};
}

// Writes the result of a probed step's selection into the layer's record and plans the next one (one thread).
__device__ __forceinline__ void select_publish(const TensorDesc& td, LayerDev& ls, const FinishIn& in, uint32_t theta, uint32_t nnz,
                                               float beta_h) {
  const uint32_t prev = in.theta_key_last;
  const uint32_t have = in.n_theta;
  ls.theta_key = theta;
  ls.theta = u2f(theta);
  ls.nnz = nnz;
  ls.sel_passes = in.passes - 1 + (in.mask_done ? 0u : 1u);  // passes over h beyond the EMA pass
  ls.probes_seen = in.probes_seen + 1;
  // ---- plan the next probed step ----
  // Two predictors of the next threshold are tracked by the error each made for this step:
  // "hold" (the last threshold; best when the threshold only jitters) and a damped extrapolation
  // in the value domain, theta + r (theta - prev), best while the curvature EMA still settles:
  // the distance of the threshold from its limit then shrinks by a nearly constant factor per
  // probe, so r is the ratio of the last two differences, kept within [0, 1] (between "hold" and
  // a straight line), and beta_h, the factor by which the EMA forgets, while only two thresholds
  // are known.  Each predictor keeps a running mean of its squared error in keys (an error three
  // times the running deviation replaces the mean at once); the one with the smaller mean is
  // used, and the band is a multiple of its deviation.
  const uint32_t prev2 = in.theta_key_last2;
  const float unknown2 = (float)kUnknownPredErr * (float)kUnknownPredErr;
  auto track = [](float var, float err, bool first) {
    const float e2 = err * err;
    if (first || e2 > 9.0f * var) return e2;
    return 0.75f * var + 0.25f * e2;
  };
  float v_hold = unknown2, v_ext = in.pred_ext_key ? in.var_ext : 3.0e38f;
  if (have >= 1) v_hold = track(in.var_hold, (float)abs_diff(theta, prev), have < 2);
  if (in.pred_ext_key) v_ext = track(v_ext, (float)abs_diff(theta, in.pred_ext_key), !(v_ext < 3.0e38f));
  if (in.window_missed) {
    v_hold = fmaxf(v_hold, unknown2);
    if (v_ext < 3.0e38f) v_ext = fmaxf(v_ext, unknown2);
  }
  uint32_t ext = 0;
  if (have >= 1) {
    const double v0 = (double)u2f(theta), v1 = (double)u2f(prev);
    const double d1 = v0 - v1;
    double r = (double)beta_h;
    if (have >= 2) {
      const double d0 = v1 - (double)u2f(prev2);
      r = d0 != 0.0 ? d1 / d0 : 1.0;
    }
    r = fmin(fmax(r, 0.0), 1.0);
    const float p = (float)(v0 + r * d1);
    ext = p > 0.0f ? min(max(f2u(p), 1u), 0x7f7fffffu) : 1u;
  }
  ls.var_hold = v_hold;
  ls.var_ext = v_ext;
  ls.pred_ext_key = ext;
  ls.theta_key_last2 = prev;
  ls.theta_key_last = theta;
  ls.n_theta = have < 2 ? have + 1 : 2;
  const bool extrapolate = ext != 0u && v_ext < v_hold;
  // e: 1.5 deviations of the chosen predictor (band = 3 e = 4.5 deviations, window half = 32 e)
  const float dev = 1.5f * sqrtf(extrapolate ? v_ext : v_hold);
  const uint32_t e = dev < 16.0f ? 16u : (dev > 1.0e9f ? 1000000000u : (uint32_t)dev);
  int64_t centre = extrapolate ? (int64_t)ext : (int64_t)theta;
  if (centre < 1) centre = 1;
  if (centre > 0x7f7fffff) centre = 0x7f7fffff;
  // fallback window: 2048 bins whose half (1024 bins) spans 32 e
  uint32_t s = kMinPredShift;
  while (s < kFullShift && ((uint64_t)1024 << s) < (uint64_t)32 * e) ++s;
  const uint32_t cbin = (uint32_t)centre >> s;
  const uint32_t lo_bin = cbin > (uint32_t)(kHistBins / 2) ? cbin - kHistBins / 2 : 0u;
  // band: 3 e on either side of the centre
  const uint64_t half = (uint64_t)3 * e;
  const uint32_t band_lo = (uint64_t)centre > half ? (uint32_t)((uint64_t)centre - half) : 1u;
  const uint64_t hi64 = (uint64_t)centre + half + 1;
  const uint32_t band_hi = hi64 < 0x7f800000ull ? (uint32_t)hi64 : 0x7f800000u;
  // expected number of keys inside the band, from the key density around this step's threshold;
  // listing them only pays when they fit the lists with room to spare
  const uint64_t expect = in.dens_width ? ((uint64_t)(band_hi - band_lo) * in.dens_count) / in.dens_width : 0u;
  ls.mode = kSelHist;
  ls.win_lo = lo_bin << s;
  ls.win_hi = ls.win_lo + ((uint32_t)kHistBins << s);
  ls.win_shift = s;
  ls.win_bins = kHistBins;
  ls.band_lo = band_lo;
  ls.band_hi = band_hi;
  ls.use_band = expect <= (uint64_t)(td.cand_cap - td.cand_cap / 4) ? 1u : 0u;
  ls.predicted = 1;
  ls.window_missed = 0;
  ls.mask_done = 0;
  ls.passes = 0;
  ls.above = 0;
  ls.k_rem = 0;
  ls.sel_count = 0;
  ls.dens_count = 0;
  ls.dens_width = 0;
  ls.acc_above = 0;
}

// Shared memory of the histogram functions, for a workgroup of kThreads threads.
struct HistShared {
  uint32_t hist[kHistBins];
  uint32_t part[kThreads / kWave];
  uint32_t out[8];
};

// Shared memory of select_finish, for a workgroup of NT threads.
template <int NT>
struct SelectShared {
  uint32_t hist[kHistBins];
  uint32_t part[NT / kWave];
  uint32_t out[8];
  uint32_t kept;
  uint32_t counts[kCandLists + 1];
  uint32_t prefix[kCandLists + 2];
};

// The whole workgroup (NT threads) calls it for tensor l, whose threshold is exact or confined to a range
// whose keys are all listed (ls.mode).  Up to REGS listed keys per thread are held in registers.
// `listed` is this thread's list length (threads 0 .. kCandLists), read ahead together with `in`.
template <int NT, int REGS>
__device__ __forceinline__ void select_finish(uint32_t l, const TensorDesc& td, LayerDev& ls, const FinishIn& in,
                                              uint32_t listed, const Candidate* cands, uint32_t* counters, float beta_h,
                                              SelectShared<NT>& sh) {
  uint32_t* const s_hist = sh.hist;
  uint32_t* const s_counts = sh.counts;
  uint32_t* const s_prefix = sh.prefix;
  // lengths and exclusive prefix sums of the lists (flat numbering of the listed keys)
  static_assert(kCandLists == kWave, "one lane per sub-list");
  if (threadIdx.x <= kCandLists) s_counts[threadIdx.x] = min(listed, threadIdx.x < kCandLists ? td.sub_cap : td.cand_cap);
  if (threadIdx.x < kWave) {
    const uint32_t incl = wave_scan(min(listed, td.sub_cap));
    if (threadIdx.x == 0) {
      s_prefix[0] = 0;
      sh.kept = 0;
    }
    s_prefix[threadIdx.x + 1] = incl;
  }
  __syncthreads();
  if (threadIdx.x == 0) s_prefix[kCandLists + 1] = s_prefix[kCandLists] + s_counts[kCandLists];
  __syncthreads();
  const uint32_t mode = in.mode;
  const uint32_t above = in.above;
  const uint32_t rng_lo = in.rng_lo, rng_hi = in.rng_hi;
  uint32_t theta = in.theta_key;
  uint32_t nnz = above + in.sel_count;
  if (mode == kSelExact && theta == 0u) nnz = in.nonzero;
  if (mode == kSelCand) {
    // all listed keys lie in [rng_lo, rng_hi); select inside the enclosing power-of-two range
    uint32_t lo = rng_lo;
    const uint32_t width = rng_hi - rng_lo;
    uint32_t width_shift = 32u - (uint32_t)__clz(width - 1u);  // ceil(log2(width)), width >= 2
    if (width <= 1u) width_shift = 0;
    uint32_t r = in.k_rem - above;
    const uint32_t inside = s_prefix[kCandLists + 1];
    // up to REGS keys per thread are held in registers for the passes below; longer lists
    // are re-read from memory in every pass
    const bool in_regs = inside <= (uint32_t)(NT * REGS);
    Candidate reg[REGS];
    uint32_t have = 0;
    if (in_regs) {
#pragma unroll
      for (int i = 0; i < REGS; ++i) {
        const uint32_t f = (uint32_t)i * NT + threadIdx.x;
        reg[i] = Candidate{0u, 0u};
        if (f < inside) {
          uint32_t a = 0, b = kCandLists + 1;  // s_prefix[a] <= f < s_prefix[b]
          while (b - a > 1) {
            const uint32_t m = (a + b) >> 1;
            if (s_prefix[m] <= f) a = m;
            else b = m;
          }
          reg[i] = cands[td.cand_offset + (size_t)a * td.sub_cap + (f - s_prefix[a])];
          have |= 1u << i;
        }
      }
    }
    auto visit = [&](auto f) {
      if (in_regs) {
#pragma unroll
        for (int i = 0; i < REGS; ++i)
          if (have & (1u << i)) f(reg[i]);
      } else {
        for_each_candidate<NT>(td, cands, s_counts, f);
      }
    };
    if (r > inside) {
      theta = 0;  // fewer non-zero keys than k (small tensors only): keep every non-zero entry
    } else {
      while (width_shift > 0) {
        const uint32_t ns = width_shift > (uint32_t)kHistBits ? width_shift - kHistBits : 0u;
        const uint32_t bins = 1u << (width_shift - ns);
        for (uint32_t b = threadIdx.x; b < bins; b += NT) s_hist[b] = 0;
        __syncthreads();
        visit([&](const Candidate& c) {
          if (c.key >= lo && ((uint64_t)(c.key - lo) >> width_shift) == 0u) atomicAdd(&s_hist[(c.key - lo) >> ns], 1u);
        });
        __syncthreads();
        const BinHit hit = find_rank_from_top<NT>(s_hist, bins, r, sh.part, sh.out);
        r -= hit.higher;
        lo += hit.bin << ns;
        width_shift = ns;
      }
      theta = lo;
    }
    // listed keys had their bits left clear: set those at or above theta
    uint32_t kept = 0;
    visit([&](const Candidate& c) {
      if (c.key >= theta) {
        atomicOr(&td.mask[c.idx >> 5], 1u << (c.idx & 31u));
        ++kept;
      }
    });
    kept = wave_sum(kept);
    if ((threadIdx.x & (kWave - 1)) == 0 && kept) atomicAdd(&sh.kept, kept);
    __syncthreads();
    nnz = above + sh.kept;
  }
  __syncthreads();
  reset_cand_counters(counters, l);
  if (threadIdx.x == 0) select_publish(td, ls, in, theta, nnz, beta_h);
}

}  // namespace triaccel
