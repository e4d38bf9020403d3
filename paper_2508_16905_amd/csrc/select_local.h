// Threshold resolution inside the update's launch, on sets bound by their launches: one workgroup of kThreads
// threads per tensor, in the grid ahead of the chunks' workgroups.
#pragma once
#include "layer_body.h"

namespace triaccel {

// Keys a thread holds in registers: the two chunks of a small tensor, whole, or this many listed keys of a larger one
// with their places.
constexpr int kLocalKeys = 2 * kRows * kVec;
constexpr int kLocalListed = 16;
static_assert(kThreads * kLocalKeys >= (int)kListAllMax, "a small tensor is held in registers");

struct alignas(16) LocalSelectShared {
  uint32_t hist[kHistBins];
  uint32_t part[kThreads / kWave];
  uint32_t out[8];
  uint32_t counts[kCandLists + 1];
  uint32_t prefix[kCandLists + 2];
  uint32_t few[kWave];
  uint32_t n_few, kept;
};

// Sums of a tensor's curvature records, over the workgroup (layer_reduce without the moments).
__device__ __forceinline__ EmaTotals ema_totals(const TensorDesc& td, const EmaPartial* __restrict__ ema_partials, LayerShared& sh) {
  const EmaPartial* const q = ema_partials + td.first_chunk;
  EmaTotals e{0, 0, 0, 0, 0};
#pragma unroll 4
  for (uint32_t c = threadIdx.x; c < td.n_chunks; c += kThreads) {
    const EmaPartial x = q[c];
    e.above += x.above_zeros & 0xffffu;
    e.zeros += x.above_zeros >> 16;
    e.maxkey = max(e.maxkey, x.maxkey);
    e.listed += x.listed;
  }
  e.above = wave_sum(e.above);
  e.zeros = wave_sum(e.zeros);
  e.maxkey = wave_max(e.maxkey);
  e.listed = wave_sum(e.listed);
  const int wave = threadIdx.x / kWave;
  if ((threadIdx.x & (kWave - 1)) == 0) {
    sh.red[0][wave] = e.above;
    sh.red[1][wave] = e.zeros;
    sh.red[2][wave] = e.maxkey;
    sh.red[3][wave] = e.listed;
    sh.red[4][wave] = 0;
  }
  __syncthreads();
  return layer_ema(sh);
}

// The r-th largest of the workgroup's keys in [lo, lo + 2^shift), by histograms in LDS; as soon as the bin that holds it
// has at most 64 keys, they are collected and every wavefront compares each with all.  One histogram normally does
// (2048 bins over a predicted band, or over the two octaves below the largest key).  Returns false, and nothing else
// happens, if there are fewer than r such keys (`check`; r is at least 1).
// Only the first `used` keys of every thread are looked at (uniform): one that no thread holds costs five instructions
// and a branch all the same.
template <int KEYS>
__device__ __forceinline__ bool rank_select(const uint32_t (&key)[KEYS], uint32_t used, uint32_t lo, uint32_t shift, uint32_t r,
                                            bool check, LocalSelectShared& sh, uint32_t& theta) {
  const auto each_inside = [&](uint32_t from, uint32_t width_shift, auto f) {
#pragma unroll
    for (int i = 0; i < KEYS; ++i)
      if ((uint32_t)(i & ~3) < used)
        if (key[i] >= from && ((key[i] - from) >> width_shift) == 0u) f(key[i]);
  };
  for (;;) {
    const uint32_t ns = shift > (uint32_t)kHistBits ? shift - kHistBits : 0u;
    const uint32_t bins = 1u << (shift - ns);
    for (uint32_t b = threadIdx.x * 4; b < kHistBins; b += kThreads * 4) *reinterpret_cast<v4u*>(&sh.hist[b]) = v4u{0, 0, 0, 0};
    if (threadIdx.x == 0) sh.n_few = 0;
    __syncthreads();
    each_inside(lo, shift, [&](uint32_t k) { atomicAdd(&sh.hist[(k - lo) >> ns], 1u); });
    __syncthreads();
    const BinHit hit = find_rank_from_top<kThreads>(sh.hist, bins, r, sh.part, sh.out);
    if (check) {
      uint32_t in_window = 0;
#pragma unroll
      for (int w = 0; w < kThreads / kWave; ++w) in_window += sh.part[w];
      if (uniform(in_window) < r) return false;
      check = false;
    }
    r -= uniform(hit.higher);
    lo += uniform(hit.bin) << ns;
    shift = ns;
    if (shift == 0) {
      theta = lo;
      return true;
    }
    if (uniform(hit.count) > (uint32_t)kWave) continue;
    each_inside(lo, shift, [&](uint32_t k) { sh.few[atomicAdd(&sh.n_few, 1u)] = k; });
    __syncthreads();
    const uint32_t n = uniform(sh.n_few), lane = threadIdx.x & (kWave - 1);
    const uint32_t mine = lane < n ? sh.few[lane] : 0u;
    uint32_t larger = 0, same = 0;
    for (uint32_t j = 0; j < n; ++j) {
      const uint32_t other = (uint32_t)__builtin_amdgcn_readlane((int)mine, (int)j);
      larger += other > mine ? 1u : 0u;
      same += other == mine ? 1u : 0u;
    }
    const unsigned long long is = __ballot(lane < n && larger < r && r <= larger + same);
    theta = (uint32_t)__builtin_amdgcn_readlane((int)mine, (int)__builtin_ctzll(is));
    return true;
  }
}

// One workgroup settles tensor l if its listed keys, or its own if it is small, settle the threshold.  A tensor of
// up to kListAllMax elements is read whole, chunk by chunk as the curvature kernel wrote it (which lists nothing of it
// and leaves its mask to this function); of a larger one the keys of the band are listed.  More of these than the
// registers hold are left to k_select_tail, and so are tensors that need histograms over h; both (in k_decide_select the
// first) are noted for the next probed step, which leaves everything to that launch (`late`: this is such a step) if the
// set is within kLateChunks or kLateTensors.
//
// Beside the streaming workgroups every dependent access takes about 3 us instead of 0.7, so there are few of them:
// tables, records and list lengths; keys; then only stores.  (An earlier form with lists re-read in every pass took 100
// to 200 us in this place.)
__device__ __forceinline__ void select_local(uint32_t l, const StepTables& tab, const TensorDesc* __restrict__ tds, GlobalDev* glob,
                                             const StepScalars& sc, const Hyper& hp, LayerShared& shl, LocalSelectShared& sh) {
  const EmaPartial* const ema_partials = tab.ema_partials;
  const Candidate* const cands = tab.cands;
  uint32_t* const counters = tab.cand_counters;
  const uint64_t skip_epoch = glob->skip_epoch;
  const uint32_t late = glob->select_late;
  const TensorDesc td = tds[l];
  LayerDev& ls = tab.layers[l];
  const SelNow now = tab.inputs[l].plan;
  FinishIn in = finish_in(ls);
  uint32_t listed_here = 0;
  if (threadIdx.x <= kCandLists) listed_here = *cand_counter(counters, l, threadIdx.x);
  TA_LOADED("s"(td.mask), "s"(td.curv), "s"(td.numel), "s"(td.has_probe), "s"(td.list_all), "s"(td.first_chunk), "s"(td.n_chunks),
            "s"(now.use_band), "s"(now.band_lo), "s"(in.probes_seen), "s"(in.var_hold), "s"(late));
  if (skip_epoch == sc.step_id || !td.has_probe) return;
  const uint32_t k = topk_count(td.numel, hp.sparsity_ppm, hp.topk_abs);
  uint32_t theta = 0, nnz = 0, above = 0;
  if (threadIdx.x == 0) sh.kept = 0;
  EmaTotals e;
  if (td.list_all && !late) {
    // the tail's key first, then the rows of the two chunks
    uint32_t key[4 + kLocalKeys];
    uint32_t (&h0)[kRows][4] = *reinterpret_cast<uint32_t(*)[kRows][4]>(&key[4]);
    uint32_t (&h1)[kRows][4] = *reinterpret_cast<uint32_t(*)[kRows][4]>(&key[4 + kRows * 4]);
    const int32_t left0 = chunk_left(0, td.numel), left1 = td.numel > kChunk ? chunk_left(kChunk, td.numel) : 0;
    const Tail tail0 = tail_of(left0, threadIdx.x), tail1 = tail_of(left1, threadIdx.x);
    uint32_t tail = load_chunk<4>(td.curv, left0, tail0, h0);
    tail |= load_chunk<4>(chunk_of<4>(static_cast<const void*>(td.curv), kChunk), left1, tail1, h1);  // of one of the two
    key[0] = tail;
    key[1] = key[2] = key[3] = 0;
    const uint32_t used = 4u + 4u * (((uint32_t)td.numel + kRowElems - 1u) / kRowElems);
    e = ema_totals(td, ema_partials, shl);
#pragma unroll
    for (int i = 0; i < 4 + kLocalKeys; ++i) key[i] &= 0x7fffffffu;
    const uint32_t nonzero = (uint32_t)td.numel - e.zeros;
    if (k <= nonzero) {
      const uint32_t span = (uint32_t)kHistBins << kFirstShift;
      const bool low = e.maxkey < span;
      // keys are at least 1 here, and none exceeds the largest
      if (!rank_select(key, used, low ? 1u : e.maxkey + 1u - span, kHistBits + kFirstShift, k, true, sh, theta))
        rank_select(key, used, 1u, 31u, k, false, sh, theta);
    }
    const uint32_t from = max(theta, 1u);
    uint32_t f0 = 0, f1 = 0;
#pragma unroll
    for (int i = 0; i < kRows * 4; ++i) {
      f0 |= key[4 + i] >= from ? 1u << i : 0u;
      f1 |= key[4 + kRows * 4 + i] >= from ? 1u << i : 0u;
    }
    if (key[0] >= from) {
      if (tail0.mine) f0 |= kTailFlag;
      else f1 |= kTailFlag;
    }
    store_mask_flags(td, 0, f0, tail0);
    if (left1 > 0) store_mask_flags(td, kChunk, f1, tail1);
    const uint32_t kept = wave_sum((uint32_t)(__popc(f0) + __popc(f1)));
    __syncthreads();
    if ((threadIdx.x & (kWave - 1)) == 0) atomicAdd(&sh.kept, kept);
  } else {
    e = ema_totals(td, ema_partials, shl);
    const bool listed = select_outcome(td, now, e, k) == kOutListed;
    const bool fits = listed && e.listed <= (uint32_t)(kThreads * kLocalListed);  // (if so, no list has dropped a key)
    if (!fits || late) {
      if (threadIdx.x == 0) {
        if (!fits && !td.list_all && (listed || hp.elementwise != 1)) glob->late_epoch = sc.step_id;
        if (listed) {
          select_setup(td, ls, glob, now, e, k, kOutListed, sc.step_id);
          // (only looked at for being zero; an atomic add takes 20 ns, one after the other for all tensors of a late step)
          glob->mask_pending[sc.step_id & 1u] = 1;
        }
      }
      return;
    }
    // lengths and first places of the lists in a flat numbering of the listed keys
    if (threadIdx.x <= kCandLists) sh.counts[threadIdx.x] = min(listed_here, threadIdx.x < kCandLists ? td.sub_cap : td.cand_cap);
    if (threadIdx.x < kWave) {
      const uint32_t incl = wave_scan(min(listed_here, td.sub_cap));
      if (threadIdx.x == 0) sh.prefix[0] = 0;
      sh.prefix[threadIdx.x + 1] = incl;
    }
    __syncthreads();
    const uint32_t inside = e.listed;
    uint32_t key[kLocalListed], idx[kLocalListed];
#pragma unroll
    for (int i = 0; i < kLocalListed; ++i) {
      key[i] = idx[i] = 0;
      if ((uint32_t)(i * kThreads) < inside) {
        const uint32_t f = (uint32_t)i * kThreads + threadIdx.x;
        if (f < inside) {
          uint32_t a = 0, b = kCandLists + 1;  // prefix[a] <= f < prefix[b]
          while (b - a > 1) {
            const uint32_t m = (a + b) >> 1;
            if (sh.prefix[m] <= f) a = m;
            else b = m;
          }
          const Candidate c = cands[td.cand_offset + (size_t)a * td.sub_cap + (f - sh.prefix[a])];
          key[i] = c.key;
          idx[i] = c.idx;
        }
      }
    }
    const uint32_t width = now.band_hi - now.band_lo;
    above = e.above;
    // band_lo is at least 1: a place without a key is in no range
    rank_select(key, (inside + kThreads - 1) / kThreads, now.band_lo, width > 1u ? 32u - (uint32_t)__clz(width - 1u) : 0u, k - above, false, sh, theta);
    // listed keys had their bits left clear: set those at or above theta
    uint32_t kept = 0;
#pragma unroll
    for (int i = 0; i < kLocalListed; ++i) {
      if ((uint32_t)(i * kThreads) < inside && key[i] >= theta) {
        atomicOr(&td.mask[idx[i] >> 5], 1u << (idx[i] & 31u));
        ++kept;
      }
    }
    kept = wave_sum(kept);
    if ((threadIdx.x & (kWave - 1)) == 0 && kept) atomicAdd(&sh.kept, kept);
    reset_cand_counters(counters, l);
    in.dens_count = e.listed;
    in.dens_width = width;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  nnz = above + sh.kept;
  in.passes = in.mask_done = 1;
  ls.nonzero = (uint32_t)td.numel - e.zeros;
  ls.sel_listed = td.list_all ? ls.nonzero : e.listed;
  ls.sel_outcome = td.list_all ? 0u : 1u;
  ls.acc_maxkey = e.maxkey;
  select_publish(td, ls, in, theta, nnz, hp.beta_curv);
}

}  // namespace triaccel
