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
//   * Tensors with at most kListAllMax elements list all their non-zero keys and select from the list.
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

template <bool FULL>
__device__ __forceinline__ void hist_chunk(const TensorDesc& td, int64_t base, const Window& w, uint32_t* s_hist,
                                           bool count_above, uint32_t& above) {
  const int tid = threadIdx.x;
  float h[kRows][4];
#pragma unroll
  for (int r = 0; r < kRows; ++r) {
    const int64_t idx = base + r * kRowElems + tid * kVec;
    if (FULL) load4<kFP32>(td.curv, idx, h[r]);
    else load4_guard<kFP32>(td.curv, idx, td.numel, 0.0f, h[r]);
  }
#pragma unroll
  for (int r = 0; r < kRows; ++r) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t key = f2u(h[r][i]) & 0x7fffffffu;  // guarded fill 0 is never counted
      if (key != 0u && key >= w.lo) {
        if (key < w.hi) atomicAdd(&s_hist[(key - w.lo) >> w.shift], 1u);
        else if (count_above) ++above;
      }
    }
  }
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
  // level 0: every thread sums its run of bins; level 1: every lane of wavefront 0 sums a run of
  // thread sums; a suffix scan over the 64 lanes locates the lane, then the thread, then the bin.
  constexpr int G = NT / kWave;  // thread sums per lane of wavefront 0
  const uint32_t per = (bins + NT - 1) / NT;
  const uint32_t b0 = threadIdx.x * per;
  uint32_t sum = 0;
  for (uint32_t b = b0; b < min(b0 + per, bins); ++b) sum += s_hist[b];
  s_part[threadIdx.x] = sum;
  __syncthreads();
  if (threadIdx.x < kWave) {
    const int lane = threadIdx.x;
    uint32_t mine = 0;
#pragma unroll
    for (int i = 0; i < G; ++i) mine += s_part[lane * G + i];
    uint32_t suffix = mine;  // sum over lanes >= this one
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const uint32_t t = __shfl_down(suffix, o);
      if (lane + o < kWave) suffix += t;
    }
    const unsigned long long reach = __ballot(suffix >= r);  // lanes from which the top reaches rank r
    const int pick = reach ? 63 - __clzll(reach) : 0;         // the highest such lane holds the rank
    if (lane == pick) {
      uint32_t acc = suffix - mine;  // keys in lanes above
      int t = pick * G + G - 1;
      for (; t > pick * G; --t) {
        if (acc + s_part[t] >= r) break;
        acc += s_part[t];
      }
      s_out[0] = (uint32_t)t;
      s_out[1] = acc;
    }
  }
  __syncthreads();
  if (threadIdx.x == s_out[0]) {
    uint32_t acc = s_out[1];
    uint32_t b = min(b0 + per, bins);
    uint32_t found = b0, cnt = 0;
    while (b > b0) {
      --b;
      const uint32_t v = s_hist[b];
      if (acc + v >= r) {
        found = b;
        cnt = v;
        break;
      }
      acc += v;
    }
    s_out[2] = found;
    s_out[3] = acc;
    s_out[4] = cnt;
  }
  __syncthreads();
  BinHit hit{s_out[2], s_out[3], s_out[4]};
  __syncthreads();
  return hit;
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
      if (b2 + kChunk <= td.numel) hist_chunk<true>(td, b2, w2, s_hist, false, unused);
      else hist_chunk<false>(td, b2, w2, s_hist, false, unused);
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

// Sum of a per-thread count over the workgroup (NT threads); s_red holds one word per wavefront.
template <int NT>
__device__ __forceinline__ uint32_t finish_block_sum(uint32_t v, uint32_t* s_red) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & (kWave - 1)) == 0) s_red[threadIdx.x / kWave] = v;
  __syncthreads();
  uint32_t t = 0;
#pragma unroll
  for (int w = 0; w < NT / kWave; ++w) t += s_red[w];
  return t;
}

// Shared memory of the histogram functions, for a workgroup of kThreads threads.
struct HistShared {
  uint32_t hist[kHistBins];
  uint32_t part[kThreads];
  uint32_t out[8];
};

// Shared memory of select_finish, for a workgroup of NT threads.
template <int NT>
struct SelectShared {
  uint32_t hist[kHistBins];
  uint32_t part[NT];
  uint32_t red[NT / kWave];
  uint32_t out[8];
  uint32_t counts[kCandLists + 1];
  uint32_t prefix[kCandLists + 2];
};

// The whole workgroup (NT threads) calls it for tensor l, whose threshold is exact or confined to a range
// whose keys are all listed (ls.mode).  Up to REGS listed keys per thread are held in registers.
template <int NT, int REGS>
__device__ __forceinline__ void select_finish(uint32_t l, const TensorDesc& td, LayerDev& ls, const Candidate* cands,
                              uint32_t* counters, float beta_h, SelectShared<NT>& sh) {
  uint32_t* const s_hist = sh.hist;
  uint32_t* const s_part = sh.part;
  uint32_t* const s_red = sh.red;
  uint32_t* const s_out = sh.out;
  uint32_t* const s_counts = sh.counts;
  uint32_t* const s_prefix = sh.prefix;
  if (threadIdx.x <= kCandLists) {
    const uint32_t c = *cand_counter(counters, l, threadIdx.x);
    s_counts[threadIdx.x] = min(c, threadIdx.x < kCandLists ? td.sub_cap : td.cand_cap);
  }
  __syncthreads();
  const uint32_t mode = ls.mode;
  const uint32_t above = ls.above;
  const uint32_t rng_lo = ls.rng_lo, rng_hi = ls.rng_hi;
  uint32_t theta = ls.theta_key;
  uint32_t nnz = above + ls.sel_count;
  if (mode == kSelExact && theta == 0u) nnz = ls.nonzero;
  if (mode == kSelCand) {
    // all listed keys lie in [rng_lo, rng_hi); select inside the enclosing power-of-two range
    uint32_t lo = rng_lo;
    const uint32_t width = rng_hi - rng_lo;
    uint32_t width_shift = 32u - (uint32_t)__clz(width - 1u);  // ceil(log2(width)), width >= 2
    if (width <= 1u) width_shift = 0;
    uint32_t r = ls.k_rem - above;
    // exclusive prefix sums of the list lengths (flat numbering of the listed keys)
    static_assert(kCandLists == kWave, "one lane per sub-list");
    if (threadIdx.x < kWave) {
      const uint32_t incl = wave_scan(s_counts[threadIdx.x]);
      if (threadIdx.x == 0) s_prefix[0] = 0;
      s_prefix[threadIdx.x + 1] = incl;
      if (threadIdx.x == kWave - 1) s_prefix[kCandLists + 1] = incl + s_counts[kCandLists];
    }
    __syncthreads();
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
        const BinHit hit = find_rank_from_top<NT>(s_hist, bins, r, s_part, s_out);
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
    kept = finish_block_sum<NT>(kept, s_red);
    nnz = above + kept;
  }
  __syncthreads();
  reset_cand_counters(counters, l);
  if (threadIdx.x != 0) return;
  // ---- publish ----
  const uint32_t prev = ls.theta_key_last;
  const uint32_t have = ls.n_theta;
  ls.theta_key = theta;
  ls.theta = u2f(theta);
  ls.nnz = nnz;
  ls.sel_passes = ls.passes - 1 + (ls.mask_done ? 0u : 1u);  // passes over h beyond the EMA pass
  ls.probes_seen = ls.probes_seen + 1;
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
  const uint32_t prev2 = ls.theta_key_last2;
  const float unknown2 = (float)kUnknownPredErr * (float)kUnknownPredErr;
  auto track = [](float var, float err, bool first) {
    const float e2 = err * err;
    if (first || e2 > 9.0f * var) return e2;
    return 0.75f * var + 0.25f * e2;
  };
  float v_hold = unknown2, v_ext = ls.pred_ext_key ? ls.var_ext : 3.0e38f;
  if (have >= 1) v_hold = track(ls.var_hold, (float)abs_diff(theta, prev), have < 2);
  if (ls.pred_ext_key) v_ext = track(v_ext, (float)abs_diff(theta, ls.pred_ext_key), !(v_ext < 3.0e38f));
  if (ls.window_missed) {
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
  const uint64_t expect = ls.dens_width ? ((uint64_t)(band_hi - band_lo) * ls.dens_count) / ls.dens_width : 0u;
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


}  // namespace triaccel
