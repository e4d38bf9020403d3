// gfx950 kernels of the Tri-Accel optimizer step.
//
// Every kernel streams tensors in chunks of kChunk = 4096 elements: four rows of 256 lanes, each
// lane holding 4 consecutive elements (one 128-bit access per lane, row and fp32 array).  All
// arithmetic that decides a stored value is fp32 with an explicit operation order (fmaf where a
// fused multiply-add is meant; the file is compiled with -ffp-contract=off); reductions are fp64.
#include "layer_body.h"

namespace triaccel {

// ---------------------------------------------------------------------------------------------
// Stage 1: per-chunk gradient moments and non-finite scan (Sec. 3.1, Var[grad_l(t)]).
// One workgroup per chunk.  Each lane accumulates, in fp64, the sums of (x - K) and (x - K)^2 of
// its 16 unscaled values x = fp32(g) * inv_scale, where the shift K is the chunk's first value
// (a sample of the data, so the sums stay small against their cancellation).  Lanes and
// wavefronts are added in a fixed order; one (mean, M2) partial per chunk.
// ---------------------------------------------------------------------------------------------
// A lane's sums over its elements.
struct StatSums {
  double shift, s1, s2;
  uint32_t bad;
};
// `g`, `gt`: the chunk's gradients as loaded (widened in place); `first`: its first value.
template <int GD>
__device__ __forceinline__ StatSums stats_sums(uint32_t (&g)[kRows][4], uint32_t gt, float first, int32_t left, const Tail& tail,
                                               float inv_scale) {
  double s1 = 0.0, s2 = 0.0;
  const double shift = (double)(first * inv_scale);
  const auto add = [&](uint32_t bits, bool inside) {
    double d = (double)(u2f(bits) * inv_scale) - shift;
    if (!inside) d = 0.0;
    s1 += d;
    s2 = fma(d, d, s2);
  };
  if (left == kChunk) {
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      widen4<GD>(g[r]);
#pragma unroll
      for (int i = 0; i < 4; ++i) add(g[r][i], true);
    }
  } else {
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      widen4<GD>(g[r]);
#pragma unroll
      for (int i = 0; i < 4; ++i) add(g[r][i], r * kRowElems + (int)threadIdx.x * kVec + 4 <= left);
    }
    if (tail.any) add(widen1<GD>(gt), tail.mine);
  }
  // One element that is not finite, or a shift, leaves a sum that is not (x = g / S of an infinity or NaN is one too), so
  // the elements' bits are only looked at behind such a sum: three instructions fewer per element (40 tensors of 60 M, bf16, no
  // probe, 155.0 -> 152.8 us a step; of 12 M 38.3 -> 38.0).
  uint32_t bad = 0;
  if (__any(((uint32_t)__double2hiint(s1) & 0x7ff00000u) == 0x7ff00000u)) {
    const auto scan = [&](uint32_t bits) { bad |= ((bits & 0x7f800000u) == 0x7f800000u) ? 1u : 0u; };
#pragma unroll
    for (int r = 0; r < kRows; ++r)
#pragma unroll
      for (int i = 0; i < 4; ++i) scan(g[r][i]);
    if (tail.any) scan(widen1<GD>(gt));
  }
  return StatSums{shift, s1, s2, bad};
}

template <int GD, bool KEEP>
__device__ __forceinline__ StatSums stats_chunk(const TensorDesc& td, int64_t base, float inv_scale) {
  uint32_t g[kRows][4];
  // the shift is read in the same batch of loads as the data: one memory latency per chunk, not two
  const float first = load1<GD>(td.grad, base);
  // the update reads the gradients again: KEEP leaves them in the caches (figures at kKeepBytes)
  const int32_t left = chunk_left(base, td.numel);
  const Tail tail = tail_of(left, threadIdx.x);
  const uint32_t gt = load_chunk<kWords<GD>, KEEP>(chunk_of<kWords<GD>>(td.grad, base), left, tail, g);
  return stats_sums<GD>(g, gt, first, left, tail, inv_scale);
}

// The wavefronts' sums, and what a non-finite element sets; then, behind a barrier, the chunk's record (one thread).
__device__ __forceinline__ void stats_reduce(const StatSums& s, double (&s_sum)[2][kThreads / kWave], LayerDev& ls, GlobalDev* glob,
                                             uint64_t step_id) {
  const double s1 = wave_sum_f64(s.s1), s2 = wave_sum_f64(s.s2);
  const uint32_t bad = wave_or(s.bad);
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  if (lane == 0) {
    s_sum[0][wave] = s1;
    s_sum[1][wave] = s2;
    if (bad) {
      atomicExch(reinterpret_cast<unsigned long long*>(&ls.found_epoch), (unsigned long long)step_id);
      atomicExch(reinterpret_cast<unsigned long long*>(&glob->skip_epoch), (unsigned long long)step_id);
    }
  }
}
__device__ __forceinline__ void stats_record(double shift, const double (&s_sum)[2][kThreads / kWave], int64_t left,
                                             StatPartial& p) {
  double t1 = s_sum[0][0], t2 = s_sum[1][0];
#pragma unroll
  for (int w = 1; w < kThreads / kWave; ++w) {
    t1 += s_sum[0][w];
    t2 += s_sum[1][w];
  }
  const double n = (double)(left < kChunk ? left : kChunk);
  const double m2 = t2 - t1 * t1 / n;
  p.mean = shift + t1 / n;
  p.m2 = m2 < 0.0 ? 0.0 : m2;  // inf and NaN (x overflowed) stay
}

template <bool KEEP>
__global__ __launch_bounds__(kThreads) void k_grad_stats(const StepTables* __restrict__ tab, const TensorDesc* __restrict__ tds,
                                                         const ChunkRef* __restrict__ chunks, GlobalDev* glob, StepScalars arg,
                                                         int local) {
  const ChunkRef cr = chunks[blockIdx.x];
  const StepScalars sc = step_scalars(arg, *tab);
  LayerDev* const layers = tab->layers;
  StatPartial* const partials = tab->partials;
  LayerIn* const inputs = tab->inputs;
  const TensorDesc td = tds[cr.tensor];
  TA_LOADED("s"(td.grad), "s"(td.numel), "s"(td.grad_dtype), "s"(td.first_chunk), "s"(layers), "s"(partials), "s"(inputs));
  // k_update_local takes the step's decisions from this copy: it writes the layers' records while it runs
  if (local && cr.index == 0 && threadIdx.x == 0) inputs[cr.tensor] = layer_in(layers[cr.tensor]);
  const int64_t base = (int64_t)cr.index * kChunk;
  StatSums sums;
  switch (td.grad_dtype) {
    case kFP32: sums = stats_chunk<kFP32, KEEP>(td, base, sc.inv_scale); break;
    case kBF16: sums = stats_chunk<kBF16, KEEP>(td, base, sc.inv_scale); break;
    default: sums = stats_chunk<kFP16, KEEP>(td, base, sc.inv_scale); break;
  }
  __shared__ double s_sum[2][kThreads / kWave];
  stats_reduce(sums, s_sum, layers[cr.tensor], glob, sc.step_id);
  __syncthreads();
  if (threadIdx.x == 0) stats_record(sums.shift, s_sum, td.numel - base, partials[td.first_chunk + cr.index]);
}

// A chunk's record: keys above the band and zero keys, largest key, keys listed, and whether a sample was not finite, of
// every lane, in a fixed order: the wavefronts' sums, then, behind a barrier, the record (one thread).
// `listed`: the wavefront's already.
__device__ __forceinline__ void ema_reduce(uint32_t above_zeros, uint32_t maxkey, uint32_t listed, bool nonfin,
                                           uint32_t (&s_red)[4][kThreads / kWave]) {
  above_zeros = wave_sum(above_zeros);  // at most 4096 + 64 (a wavefront's seventeenth elements) in either half: no carry
  maxkey = wave_max(maxkey);
  const uint32_t anynf = __any(nonfin) ? 1u : 0u;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  if (lane == 0) {
    s_red[0][wave] = above_zeros;
    s_red[1][wave] = maxkey;
    s_red[2][wave] = listed;
    s_red[3][wave] = anynf;
  }
}
__device__ __forceinline__ EmaPartial ema_record(int32_t chunk_left, const uint32_t (&s_red)[4][kThreads / kWave]) {
  uint32_t az = 0, mk = 0, ln = 0, nf = 0;
#pragma unroll
  for (int w = 0; w < kThreads / kWave; ++w) {
    az += s_red[0][w];
    mk = max(mk, s_red[1][w]);
    ln += s_red[2][w];
    nf |= s_red[3][w];
  }
  // elements past the end of the tensor were counted as zero keys
  // (the seventeenth elements are a wavefront's, of which left % 4 exist)
  const uint32_t left = (uint32_t)chunk_left, rest = left & 3u;
  const uint32_t past = kChunk - (left - rest) + (rest ? kWave - rest : 0u);
  return EmaPartial{az - (past << 16), mk, ln, nf};
}

// ---------------------------------------------------------------------------------------------
// Stage 2: curvature EMA (diagonal Hutchinson signal of Sec. 3.2), one workgroup per chunk.
// Per element, fp32:  u = (z * hz) * inv_scale;  h = u on the tensor's first probe, else
// h = fma(beta_h, h, (1 - beta_h) * u);  a non-finite u leaves h unchanged.
// The same pass writes the provisional mask, lists the keys of the band and leaves one small
// record per chunk (keys above the band, zero keys, largest key, non-finite flag); no atomics
// except the candidate appends.
// ---------------------------------------------------------------------------------------------
// SRC selects the sample: -1 = Hutchinson pair z * Hz / S; a precision code = squared unscaled
// gradient (g / S)^2 read from the gradient buffer of that precision (empirical Fisher).
//
// Keys at or above `list_hi` get their mask bit, keys in [list_lo, list_hi) are listed: the predicted
// band; [1, 2^31) for a tensor that lists every non-zero key; an empty range above all keys when the
// threshold is found by histogram passes.  The 16 elements of a lane go through the same straight line
// of selects, without a branch: with a branch per element and condition the kernel was bound by its
// instructions on sets that fit the chip at once (4.0 M parameters: 29.6 us with, 21.2 us
// without; 11.2 M: 45.2, 35.6 us).  Elements past the tensor's end read as 0, whose sample is 0 and
// whose key is 0: they only have to be taken off the count of zero keys.
//
// SD: a precision code = the pass takes the gradients' moments as well (k_stats_ema; the same as SRC if SRC is one), and
// leaves the old values of what it overwrites with `undo`.
struct EmaRanges {
  bool listing;
  uint32_t list_lo, list_hi;
};
struct EmaShared {
  uint32_t red[4][kThreads / kWave];
};
struct StatShared {
  double sum[2][kThreads / kWave];
};
template <int SRC, int SD>
__device__ __forceinline__ void ema_chunk(const TensorDesc& td, int64_t base, const StepScalars& sc, float beta_h, float omb_h,
                                          bool first, const EmaRanges& ranges, uint32_t chunk_index, uint32_t tensor,
                                          Candidate* cands, uint32_t* counters, EmaPartial* __restrict__ ema_partials,
                                          const EmaUndo& undo, StatPartial* __restrict__ partials, LayerDev* layers, GlobalDev* glob,
                                          EmaShared& sh, StatShared& sh_stats) {
  static_assert(SRC < 0 || SD < 0 || SRC == SD, "one gradient");
  constexpr bool STATS = SD >= 0;
  uint32_t maxkey = 0;
  const uint32_t tid = threadIdx.x;
  constexpr int ZW = SRC < 0 ? 4 : kWords<SRC>, GW = STATS ? kWords<SD> : 4;
  const void* const zp = chunk_of<ZW>(SRC < 0 ? static_cast<const void*>(td.z) : td.grad, base);
  const void* const hzp = chunk_of<4>(static_cast<const void*>(td.hz), base);
  const void* const gp = chunk_of<GW>(td.grad, base);
  void* const hp = chunk_of<4>(static_cast<void*>(td.curv), base);
  const int32_t left = chunk_left(base, td.numel);
  const Rows zrows = rows_of<ZW>(zp, left), hzrows = rows_of<4>(hzp, left), hrows = rows_of<4>(hp, left);
  const Rows grows = rows_of<GW>(gp, left), urows = rows_of<4>(undo.h, left);
  uint32_t z[kRows][4], hz[SRC < 0 ? kRows : 1][4], h[kRows][4], g[SRC < 0 && STATS ? kRows : 1][4];
  float g0 = 0.0f;
  if constexpr (STATS) g0 = load1<SD>(td.grad, base);
  if constexpr (STATS && SRC < 0) {
#pragma unroll
    for (int r = 0; r < kRows; ++r) load_words<GW, true>(grows, r, tid, g[r]);
  }
#pragma unroll
  for (int r = 0; r < kRows; ++r) {
    load_words<ZW, STATS && SRC >= 0>(zrows, r, tid, z[r]);
    if constexpr (SRC < 0) load_words<4>(hzrows, r, tid, hz[r]);
    load_words<4>(hrows, r, tid, h[r]);
  }
  const Tail tail = tail_of(left, tid);
  uint32_t zt = 0, hzt = 0, ht = 0, gt = 0;
  if (tail.any) {
    if constexpr (STATS && SRC < 0) gt = load_tail<GW>(gp, tail);
    zt = load_tail<ZW>(zp, tail);
    if constexpr (SRC < 0) hzt = load_tail<4>(hzp, tail);
    ht = load_tail<4>(hp, tail);
  }
  uint32_t old_mask = 0;
  if constexpr (STATS) {
    // the lanes and words of store_mask_flags: each word is read and written by one lane
    int64_t word;
    if (mask_word_of(td, base, word)) old_mask = as_global<uint32_t>(td.mask)[word];
  }
  __builtin_amdgcn_sched_barrier(0);  // all loads first
  StatSums sums;
  if constexpr (STATS) {
    if constexpr (SRC < 0) sums = stats_sums<SD>(g, gt, g0, left, tail, sc.inv_scale);
    else {
      uint32_t x[kRows][4];
#pragma unroll
      for (int r = 0; r < kRows; ++r)
#pragma unroll
        for (int i = 0; i < GW; ++i) x[r][i] = z[r][i];
      sums = stats_sums<SD>(x, zt, g0, left, tail, sc.inv_scale);
    }
  }
  // Keys >= list_hi / >= list_lo.  The flag is the sign of (bound - 1) - key (neither reaches 2^31), shifted in from the
  // right: two instructions, where a comparison takes three.  Zero keys are counted only where the smallest is one.
  // (A wavefront issues an instruction in 1.7 to 2 ns, so 100 fewer of 600 are 0.2 us of a launch that fits the chip at
  // once: 30 tensors of 0.3 M, probed, 16.5 -> 16.1 us a step, Fisher 16.0 -> 15.7; of 20 M, Fisher, 106.2 -> 105.1.)
  uint32_t hflags = 0, lflags = 0, minkey = ~0u;
  const uint32_t below_hi = ranges.list_hi - 1u, below_lo = ranges.list_lo - 1u;
  bool any_bad = false;
  const auto element = [&](uint32_t zbits, uint32_t hzbits, uint32_t& hbits) {
    float u;
    if constexpr (SRC < 0) {
      u = u2f(zbits) * u2f(hzbits);
      u = u * sc.inv_scale;
    } else {
      // x = g / S in both factors: u = x * x
      const float x = u2f(zbits) * sc.inv_scale;
      u = x * x;
    }
    const bool bad = !__builtin_isfinite(u);
    any_bad |= bad;
    const float p = omb_h * u;
    const float next = fmaf(beta_h, u2f(hbits), p);
    // u on the first probe, the average after it, the old value where the sample is not finite
    const uint32_t bits = first ? f2u(u) : f2u(next);
    hbits = bad ? hbits : bits;
  };
  const auto look = [&](uint32_t hbits) {
    const uint32_t key = hbits & 0x7fffffffu;
    maxkey = max(maxkey, key);
    minkey = min(minkey, key);
    hflags = __builtin_amdgcn_alignbit(hflags, below_hi - key, 31);
    lflags = __builtin_amdgcn_alignbit(lflags, below_lo - key, 31);
  };
#pragma unroll
  for (int r = 0; r < kRows; ++r) {
    if constexpr (SRC >= 0) widen4<SRC>(z[r]);
    if constexpr (STATS) store_words<4>(urows, r, tid, h[r]);
#pragma unroll
    for (int i = 0; i < 4; ++i) element(z[r][i], SRC < 0 ? hz[r][i] : 0u, h[r][i]);
    store_words<4>(hrows, r, tid, h[r]);
#pragma unroll
    for (int i = 0; i < 4; ++i) look(h[r][i]);
  }
  if (tail.any) {
    if constexpr (STATS) store_tail<kFP32>(undo.h, tail, ht);
    // lanes without a seventeenth element read 0 for it, like what lies past the end
    element(SRC < 0 ? zt : widen1<SRC < 0 ? kFP32 : SRC>(zt), hzt, ht);
    store_tail<kFP32>(hp, tail, ht);
    look(ht);
  } else {
    hflags <<= 1;
    lflags <<= 1;
  }
  // element 4 r + i to bit 4 r + i, the seventeenth to bit 16
  hflags = __brev(hflags) >> 15;
  lflags = __brev(lflags) >> 15;
  uint32_t zeros = 0;
  if (__any(minkey == 0u)) {
#pragma unroll
    for (int r = 0; r < kRows; ++r)
#pragma unroll
      for (int i = 0; i < 4; ++i) zeros += (h[r][i] & 0x7fffffffu) == 0u ? 1u : 0u;
    if (tail.any) zeros += (ht & 0x7fffffffu) == 0u ? 1u : 0u;
  }
  // zero keys in the high half, keys above the band in the low half
  const uint32_t above_zeros = (zeros << 16) | (uint32_t)__popc(hflags);
  const uint32_t cflags = lflags ^ hflags;  // a key at or above list_hi is above list_lo too
  // the chunk's record is made while the list's counter answers
  Appending app{0, 0, 0};
  if constexpr (STATS) {
    int64_t word;
    if (mask_word_of(td, base, word)) as_global<uint32_t>(undo.mask)[word - (base >> 5)] = old_mask;
  }
  if (ranges.listing) {
    app = append_begin(cflags, chunk_index, tensor, td, counters);
    store_mask_flags(td, base, hflags, tail);
  }
  ema_reduce(above_zeros, maxkey, app.total, any_bad, sh.red);
  if constexpr (STATS) stats_reduce(sums, sh_stats.sum, layers[tensor], glob, sc.step_id);
  __syncthreads();
  if (tid == 0) ema_partials[td.first_chunk + chunk_index] = ema_record(left, sh.red);
  if constexpr (STATS) {
    if (tid == kWave) stats_record(sums.shift, sh_stats.sum, td.numel - base, partials[td.first_chunk + chunk_index]);
  }
  if (ranges.listing) append_end(app, cflags, h, ht, tail, base, tensor, td, cands, counters);
}

// `small`: a small tensor's keys are listed, all of them, or left to select_local, which reads them where they lie.
__device__ __forceinline__ EmaRanges ema_ranges(const TensorDesc& td, bool small, uint32_t use_band, uint32_t band_lo,
                                                uint32_t band_hi) {
  const bool list_all = td.list_all != 0 && small;
  const bool listing = list_all || (td.list_all == 0 && use_band != 0);
  // band_lo >= 1 and band_hi <= 0x7f800000, so key 0 is never in a range; no key reaches 2^31
  return EmaRanges{listing, list_all ? 1u : listing ? band_lo : 0x80000000u, list_all || !listing ? 0x80000000u : band_hi};
}

// At most 6 wavefronts per SIMD: room for the loads of all rows to be under way at once.
template <bool FISHER>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4, 6))) void k_curv_ema(
    const StepTables* __restrict__ tab, const TensorDesc* __restrict__ tds, const ChunkRef* __restrict__ chunks, const GlobalDev* glob,
    StepScalars arg, int list_small) {
  __shared__ EmaShared sh;
  const ChunkRef cr = chunks[blockIdx.x];
  const StepScalars sc = step_scalars(arg, *tab);
  // the skip word travels together with the tables: its latency is not one more before the data's
  const uint64_t skip_epoch = glob->skip_epoch;
  const uint32_t late = glob->select_late;
  const float beta_h = tab->hyper.beta_curv, omb_h = 1.0f - beta_h;
  Candidate* const cands = tab->cands;
  uint32_t* const counters = tab->cand_counters;
  EmaPartial* const ema_partials = tab->ema_partials;
  const TensorDesc td = tds[cr.tensor];
  const LayerDev& ls = tab->layers[cr.tensor];
  const uint32_t probes_seen = ls.probes_seen, use_band = ls.use_band, band_lo = ls.band_lo, band_hi = ls.band_hi;
  TA_LOADED("s"(td.grad), "s"(td.z), "s"(td.hz), "s"(td.curv), "s"(td.mask), "s"(td.numel), "s"(td.grad_dtype),
            "s"(td.has_probe), "s"(td.list_all), "s"(td.first_chunk), "s"(td.cand_offset), "s"(probes_seen), "s"(use_band), "s"(band_lo),
            "s"(band_hi), "s"(late), "s"(beta_h), "s"(cands), "s"(counters), "s"(ema_partials));
  if (skip_epoch == sc.step_id || !td.has_probe) return;
  const bool first = probes_seen == 0;
  // (`late`: select_local leaves the small tensors to k_select_tail at this step, which takes them from lists)
  const EmaRanges ranges = ema_ranges(td, (list_small | (int)late) != 0, use_band, band_lo, band_hi);
  const int64_t base = (int64_t)cr.index * kChunk;
  StatShared none;
#define TA_EMA(SRC_)                                                                                                     \
  ema_chunk<SRC_, -1>(td, base, sc, beta_h, omb_h, first, ranges, cr.index, cr.tensor, cands, counters, ema_partials,    \
                      EmaUndo{nullptr, nullptr}, nullptr, nullptr, nullptr, sh, none)
  if constexpr (!FISHER) {
    TA_EMA(-1);
  } else {
    switch (td.grad_dtype) {
      case kFP32: TA_EMA(kFP32); break;
      case kBF16: TA_EMA(kBF16); break;
      default: TA_EMA(kFP16); break;
    }
  }
#undef TA_EMA
}

// ---------------------------------------------------------------------------------------------
// Stages 1 and 2 in one launch, for probed steps of short sets (kFusedChunks).  Whether the step is skipped is only known
// when the launch has ended, so every workgroup leaves the old values of the curvature and mask that it overwrites in the
// workspace, and the update puts them back if the step turns out to be skipped (ema_undo).  Whether and what a workgroup
// stores does not depend on the skip word, so what is put back is always this step's.
// Bound by latency: 4.3 us for seven workgroups, 6.4 for 79 (the two kernels one after the other 3.1 + 5.2), 8.1 for 250, three
// dependent accesses, the reductions and the end of a kernel among them; the gradients' loads go with the others'.
// ---------------------------------------------------------------------------------------------
template <bool FISHER>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4, 6))) void k_stats_ema(
    const StepTables* __restrict__ tab, const TensorDesc* __restrict__ tds, const ChunkRef* __restrict__ chunks, GlobalDev* glob,
    StepScalars arg) {
  __shared__ EmaShared sh;
  __shared__ StatShared sh_stats;
  const ChunkRef cr = chunks[blockIdx.x];
  const StepScalars sc = step_scalars(arg, *tab);
  const uint32_t late = glob->select_late;
  const float beta_h = tab->hyper.beta_curv, omb_h = 1.0f - beta_h;
  Candidate* const cands = tab->cands;
  uint32_t* const counters = tab->cand_counters;
  EmaPartial* const ema_partials = tab->ema_partials;
  LayerDev* const layers = tab->layers;
  StatPartial* const partials = tab->partials;
  LayerIn* const inputs = tab->inputs;
  float* const undo_h = tab->undo_h;
  uint32_t* const undo_mask = tab->undo_mask;
  const TensorDesc td = tds[cr.tensor];
  const LayerDev& ls = layers[cr.tensor];
  const uint32_t probes_seen = ls.probes_seen, use_band = ls.use_band, band_lo = ls.band_lo, band_hi = ls.band_hi;
  TA_LOADED("s"(td.grad), "s"(td.z), "s"(td.hz), "s"(td.curv), "s"(td.mask), "s"(td.numel), "s"(td.grad_dtype),
            "s"(td.has_probe), "s"(td.list_all), "s"(td.first_chunk), "s"(td.cand_offset), "s"(td.undo_slot), "s"(probes_seen),
            "s"(use_band), "s"(band_lo), "s"(band_hi), "s"(late), "s"(beta_h), "s"(cands), "s"(counters), "s"(ema_partials));
  // k_update_local takes the step's decisions from this copy: it writes the layers' records while it runs
  if (cr.index == 0 && threadIdx.x == 0) inputs[cr.tensor] = layer_in(ls);
  const int64_t base = (int64_t)cr.index * kChunk;
  if (td.has_probe) {
    const bool first = probes_seen == 0;
    const EmaRanges ranges = ema_ranges(td, late != 0, use_band, band_lo, band_hi);
    const EmaUndo undo = ema_undo(undo_h, undo_mask, td, base);
#define TA_EMA(SD_)                                                                                                   \
  ema_chunk<FISHER ? SD_ : -1, SD_>(td, base, sc, beta_h, omb_h, first, ranges, cr.index, cr.tensor, cands, counters, \
                                    ema_partials, undo, partials, layers, glob, sh, sh_stats)
    switch (td.grad_dtype) {
      case kFP32: TA_EMA(kFP32); break;
      case kBF16: TA_EMA(kBF16); break;
      default: TA_EMA(kFP16); break;
    }
#undef TA_EMA
    return;
  }
  StatSums sums;
  switch (td.grad_dtype) {
    case kFP32: sums = stats_chunk<kFP32, true>(td, base, sc.inv_scale); break;
    case kBF16: sums = stats_chunk<kBF16, true>(td, base, sc.inv_scale); break;
    default: sums = stats_chunk<kFP16, true>(td, base, sc.inv_scale); break;
  }
  stats_reduce(sums, sh_stats.sum, layers[cr.tensor], glob, sc.step_id);
  __syncthreads();
  if (threadIdx.x == 0) stats_record(sums.shift, sh_stats.sum, td.numel - base, partials[td.first_chunk + cr.index]);
}

// ---------------------------------------------------------------------------------------------
// Fallback radix select: histogram pass over the tensors in histogram mode, each workgroup over
// its share of the chunk list.  The workgroup that is the last to deliver its part of a tensor's
// histogram also scans it (select_scan), so no workgroup ever waits for another.  One round is
// what a tensor normally needs, and the step launches two (a window that missed, or more keys in
// the pivot bin than can be listed, needs the second).  Beyond that (a miss followed by
// refinements, heavy ties: at most four rounds in all) the workgroup that scans makes up to
// `serial_rounds` further passes over the whole tensor on its own -- slow for a large tensor, but
// rare, and it bounds the fallback to two launches.
// Leaves at once when no tensor is in histogram mode: a workgroup that sees the pending count at
// zero owns no chunk of a tensor still being counted, because a tensor's scan, which alone
// lowers the count, needs every workgroup owning one of its chunks to have arrived.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void k_hist_pass(const StepTables* __restrict__ tab, const TensorDesc* __restrict__ tds,
                                                        const ChunkRef* __restrict__ chunks, GlobalDev* glob, StepScalars arg,
                                                        int serial_rounds, uint32_t n_wg) {
  const StepScalars sc = step_scalars(arg, *tab);
  LayerDev* const layers = tab->layers;
  uint32_t* const hist = tab->hist;
  const uint32_t total_chunks = tab->total_chunks;
  const uint64_t skip_epoch = glob->skip_epoch;
  const uint32_t pending = __hip_atomic_load(&glob->hist_pending[sc.step_id & 1u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (pending == 0 || skip_epoch == sc.step_id) return;
  __shared__ uint32_t s_hist[kHistBins];
  __shared__ uint32_t s_part[kThreads / kWave];
  __shared__ uint32_t s_out[8];
  __shared__ uint32_t s_last;
  for (int b = threadIdx.x; b < kHistBins; b += kThreads) s_hist[b] = 0;
  __syncthreads();
  const uint32_t per = (total_chunks + n_wg - 1) / n_wg;
  const uint32_t c0 = min(blockIdx.x * per, total_chunks);
  const uint32_t c1 = min(c0 + per, total_chunks);
  int cur = -1;
  bool active = false;
  Window w{0, 0, 0, 0};
  TensorDesc td;
  bool count_above = false;  // the number of keys above the window is not known yet (predicted window)
  uint32_t above = 0;
  uint32_t mine = 0;         // chunks of the current tensor counted by this workgroup
  uint32_t c = c0;
  while (c <= c1) {
    const bool end = (c == c1);
    const int t = end ? -2 : (int)chunks[c].tensor;
    if (t != cur) {
      if (cur >= 0 && active) {
        flush_hist(s_hist, w.bins, hist + (size_t)cur * kHistBins);
        above = wave_sum(above);
        if ((threadIdx.x & (kWave - 1)) == 0 && above) atomicAdd(&layers[cur].acc_above, above);
        // release: this workgroup's atomics are complete before its arrival is counted
        __threadfence();
        __syncthreads();
        if (threadIdx.x == 0) {
          const uint32_t before = atomicAdd(&layers[cur].hist_arrived, mine);
          s_last = (before + mine == td.n_chunks) ? 1u : 0u;
        }
        __syncthreads();
        if (s_last) {
          __threadfence();  // acquire: the scan below reads what the other workgroups added
          select_scan((uint32_t)cur, td, layers[cur], glob, hist, sc.step_id, s_hist, s_part, s_out, true);
          select_serial((uint32_t)cur, td, layers[cur], glob, hist, sc.step_id, s_hist, s_part, s_out, serial_rounds);
          for (int b = threadIdx.x; b < kHistBins; b += kThreads) s_hist[b] = 0;
          __syncthreads();
        }
      }
      if (end) break;
      cur = t;
      td = tds[t];
      const LayerDev& ls = layers[t];
      active = td.has_probe != 0 && ls.mode == kSelHist && ls.passes > 0;
      w = Window{ls.win_lo, ls.win_shift, ls.win_bins, ls.win_hi};
      count_above = ls.count_above != 0;
      above = 0;
      mine = 0;
      if (!active) {
        // jump over the rest of this tensor's chunks owned by this workgroup
        c = min(td.first_chunk + td.n_chunks, c1);
        continue;
      }
    }
    const int64_t base = (int64_t)chunks[c].index * kChunk;
    hist_chunk(td, base, w, s_hist, count_above, above);
    ++mine;
    ++c;
  }
}

// ---------------------------------------------------------------------------------------------
// Finish (select_finish) as a kernel of its own, one workgroup per tensor.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kFinishThreads) void k_select_finish(const StepTables* __restrict__ tab,
                                                                  const TensorDesc* __restrict__ tds, const GlobalDev* glob,
                                                                  StepScalars arg) {
  __shared__ SelectShared<kFinishThreads> sh;
  const StepScalars sc = step_scalars(arg, *tab);
  LayerDev* const layers = tab->layers;
  uint32_t* const counters = tab->cand_counters;
  const uint64_t skip_epoch = glob->skip_epoch;
  const uint32_t l = blockIdx.x;
  const uint32_t listed = threadIdx.x <= kCandLists ? *cand_counter(counters, l, threadIdx.x) : 0u;
  const TensorDesc td = tds[l];
  const FinishIn in = finish_in(layers[l]);
  TA_LOADED("s"(td.mask), "s"(td.has_probe), "s"(td.cand_cap), "s"(in.mode), "s"(in.probes_seen), "s"(in.var_hold));
  if (skip_epoch == sc.step_id || !td.has_probe) return;
  select_finish<kFinishThreads, kFinishRegs>(l, td, layers[l], in, listed, tab->cands, counters, tab->hyper.beta_curv, sh);
}

// ---------------------------------------------------------------------------------------------
// Stage 4: per-layer kernel (one workgroup per tensor; sets of the local form have none): band check of the
// threshold selection (select_outcome, select_setup), then the per-layer assignment (layer_body.h), overflow
// decision and loss-scale schedule.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void k_layer(const StepTables* __restrict__ tab, const TensorDesc* __restrict__ tds,
                                                    GlobalDev* glob, StepScalars arg) {
  const StepScalars sc = step_scalars(arg, *tab);
  const Hyper hp = tab->hyper;
  const uint32_t l = blockIdx.x;
  const TensorDesc td = tds[l];
  LayerDev& ls = tab->layers[l];
  const bool skip = step_skipped(glob, sc.step_id);
  __shared__ LayerShared sh;
  LayerSums sums{};
  int outcome = kOutListed;
  const uint32_t k = topk_count(td.numel, hp.sparsity_ppm, hp.topk_abs);
  const SelNow now = select_plan(ls);
  const LayerIn in = layer_in(ls);
  if (!skip) {
    sums = layer_reduce<true>(layer_accumulate<true>(td, tab->partials, tab->ema_partials, td.has_probe != 0), td.numel, sh);
    if (td.has_probe) outcome = select_outcome(td, now, sums.ema, k);
    if (outcome != kOutListed) reset_cand_counters(tab->cand_counters, l);  // drop whatever the EMA kernel listed
  }
  if (threadIdx.x != 0) return;
  if (!skip) {
    if (td.has_probe) select_setup(td, ls, glob, now, sums.ema, k, outcome, sc.step_id);
    layer_publish(l, ls, layer_decide(in, sums, td.has_probe != 0, sc.lr, hp), glob, tab->trans_list, tab->n_tensors,
                  sc.step_id);
  } else {
    ls.found_inf = (ls.found_epoch == sc.step_id) ? 1u : 0u;
  }
  if (l == 0) step_record(glob, tab->host_result, sc, hp, skip);
}

// ---------------------------------------------------------------------------------------------
// Host-side launchers
// ---------------------------------------------------------------------------------------------
hipError_t launch_grad_stats(const DeviceTables& t, const StepScalars& sc, bool local, hipStream_t s) {
  const auto kernel = t.keep_grads ? k_grad_stats<true> : k_grad_stats<false>;
  return launch(kernel, t.total_chunks, kThreads, s, t.dev, t.tensors, t.wg_chunks, t.glob, sc, local ? 1 : 0);
}

hipError_t launch_curv_ema(const DeviceTables& t, const StepScalars& sc, bool fisher, bool local, hipStream_t s) {
  const auto kernel = fisher ? k_curv_ema<true> : k_curv_ema<false>;
  return launch(kernel, t.total_chunks, kThreads, s, t.dev, t.tensors, t.wg_chunks, t.glob, sc, local ? 0 : 1);
}

hipError_t launch_stats_ema(const DeviceTables& t, const StepScalars& sc, bool fisher, hipStream_t s) {
  const auto kernel = fisher ? k_stats_ema<true> : k_stats_ema<false>;
  return launch(kernel, t.total_chunks, kThreads, s, t.dev, t.tensors, t.wg_chunks, t.glob, sc);
}

hipError_t launch_hist_pass(const DeviceTables& t, const StepScalars& sc, int serial_rounds, hipStream_t s) {
  const uint32_t grid = t.total_chunks < t.persistent_grid ? t.total_chunks : t.persistent_grid;
  return launch(k_hist_pass, grid, kThreads, s, t.dev, t.tensors, t.chunks, t.glob, sc, serial_rounds, grid);
}

hipError_t launch_select_finish(const DeviceTables& t, const StepScalars& sc, hipStream_t s) {
  return launch(k_select_finish, t.n_tensors, kFinishThreads, s, t.dev, t.tensors, t.glob, sc);
}

hipError_t launch_layer(const DeviceTables& t, const StepScalars& sc, hipStream_t s) {
  return launch(k_layer, t.n_tensors, kThreads, s, t.dev, t.tensors, t.glob, sc);
}

}  // namespace triaccel
