// Device helpers shared by the translation units of the optimizer-step kernels: wavefront
// reductions, the mask-word gather, the candidate lists and the fallback mask pass of a chunk.
#pragma once
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "numerics.h"

namespace triaccel {

// ---------------------------------------------------------------------------------------------
// wavefront (64 lanes) helpers
// ---------------------------------------------------------------------------------------------
// Reductions and the inclusive scan over the 64 lanes move data inside the vector ALU (data-parallel
// primitives) instead of through LDS: shifts by 1, 2, 4, 8 inside the rows of 16 lanes, then the last
// lane of row 0 / 2 to row 1 / 3 (row_bcast15) and of the first half to the second (row_bcast31).
// Lanes without a source get `0`, the identity of +, | and of max over unsigned values.
#define TA_DPP(v, ctrl, rows) ((uint32_t)__builtin_amdgcn_update_dpp(0, (int)(v), (ctrl), (rows), 0xF, false))
#define TA_DPP_TREE(v, OP)                        \
  do {                                            \
    v = OP(v, TA_DPP(v, 0x111, 0xF));             \
    v = OP(v, TA_DPP(v, 0x112, 0xF));             \
    v = OP(v, TA_DPP(v, 0x114, 0xF));             \
    v = OP(v, TA_DPP(v, 0x118, 0xF));             \
    v = OP(v, TA_DPP(v, 0x142, 0xA));             \
    v = OP(v, TA_DPP(v, 0x143, 0xC));             \
  } while (0)
#define TA_OP_ADD(a, b) ((a) + (b))
#define TA_OP_OR(a, b) ((a) | (b))
#define TA_OP_MAX(a, b) (max((uint32_t)(a), (uint32_t)(b)))
__device__ __forceinline__ uint32_t last_lane(uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)v, kWave - 1); }
__device__ __forceinline__ uint32_t first_lane(uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)v, 0); }
// The same value in every lane, in a scalar register from here on.
__device__ __forceinline__ uint32_t uniform(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
template <typename T>
__device__ __forceinline__ T* uniform(T* p) {
  const uint64_t a = (uint64_t)p;
  return (T*)((uint64_t)uniform((uint32_t)(a >> 32)) << 32 | uniform((uint32_t)a));
}
// Sum over this lane and the lanes below it; all lanes of the wavefront must be active.
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
  TA_DPP_TREE(v, TA_OP_ADD);
  return v;
}
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) { return last_lane(wave_scan(v)); }
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
  TA_DPP_TREE(v, TA_OP_MAX);
  return last_lane(v);
}
__device__ __forceinline__ uint32_t wave_or(uint32_t v) {
  TA_DPP_TREE(v, TA_OP_OR);
  return last_lane(v);
}

// Sum over the 64 lanes, in a fixed order, valid in every lane.
#define TA_DPP_F64(v, ctrl, rows)                                                                          \
  __hiloint2double((int)TA_DPP((uint32_t)__double2hiint(v), ctrl, rows), (int)TA_DPP((uint32_t)__double2loint(v), ctrl, rows))
__device__ __forceinline__ double wave_sum_f64(double v) {
  v += TA_DPP_F64(v, 0x111, 0xF);
  v += TA_DPP_F64(v, 0x112, 0xF);
  v += TA_DPP_F64(v, 0x114, 0xF);
  v += TA_DPP_F64(v, 0x118, 0xF);
  v += TA_DPP_F64(v, 0x142, 0xA);
  v += TA_DPP_F64(v, 0x143, 0xC);
  return __hiloint2double((int)last_lane((uint32_t)__double2hiint(v)), (int)last_lane((uint32_t)__double2loint(v)));
}

// Set by the gradient-statistics kernel and read by the kernels after it (an ordinary load: the writer
// is an earlier kernel).
__device__ __forceinline__ bool step_skipped(const GlobalDev* glob, uint64_t step_id) { return glob->skip_epoch == step_id; }

// TA_LOADED(operands): the loads of these wave-uniform values ("s"(x), ...) are issued together and ahead of
// whatever follows.  Without it the compiler moves a load that is only used behind a branch to behind that
// branch, where its latency comes on top of that of the load that the branch waits for.
#define TA_LOADED(...) asm volatile("" ::__VA_ARGS__)

// The step's scalars: the launch's, or of a captured step the last ones that were written to device memory.  Both are
// read, without a branch.
__device__ __forceinline__ StepScalars step_scalars(const StepScalars& arg, const StepTables& tab) {
  const StepScalars dev = tab.scalars;
  const bool c = arg.captured != 0;
  return StepScalars{c ? dev.lr : arg.lr, c ? dev.loss_scale : arg.loss_scale, c ? dev.inv_scale : arg.inv_scale, 0u,
                     c ? dev.step_id : arg.step_id};
}

__device__ __forceinline__ uint32_t elem_size(int code) { return code == kFP32 ? 4u : 2u; }

// Data-parallel-primitive moves inside the wavefront (no LDS traffic): swap neighbours in a quad,
// swap the quad's halves, then mirror the 8-lane half row (lane i reads lane 7 - i; after the first
// two steps all four lanes of a quad agree, so the mirror brings in the other quad's value).
#define TA_DPP_OR(v, ctrl) ((v) | (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(v), (ctrl), 0xF, 0xF, true))
// Eight consecutive lanes hold the 32 elements of one mask word: combine their 4-bit nibbles.
__device__ __forceinline__ uint32_t gather_mask_word(uint32_t nib, int lane) {
  uint32_t v = nib << (4 * (lane & 7));
  v = TA_DPP_OR(v, 0xB1);   // quad_perm [1, 0, 3, 2]
  v = TA_DPP_OR(v, 0x4E);   // quad_perm [2, 3, 0, 1]
  v = TA_DPP_OR(v, 0x141);  // row_half_mirror
  return v;
}

// A tensor's elements from `base`, W bytes each, and their number as far as a chunk goes.
template <int W>
__device__ __forceinline__ const void* chunk_of(const void* tensor, int64_t base) {
  return static_cast<const char*>(tensor) + base * W;
}
template <int W>
__device__ __forceinline__ void* chunk_of(void* tensor, int64_t base) {
  return static_cast<char*>(tensor) + base * W;
}
static_assert(kRowLanes == kThreads && kRowElems == kRowLanes * kVec, "rows of the accessors");
__device__ __forceinline__ int32_t chunk_left(int64_t base, int64_t n) { return (int32_t)(n - base < kChunk ? n - base : kChunk); }

// The 16 elements of every lane of the chunk that starts at `chunk`, as they lie in memory, and the seventeenth of
// the lanes that have one (0 in the others).
template <int W, bool KEEP = false>
__device__ __forceinline__ uint32_t load_chunk(const void* chunk, int32_t left, const Tail& t, uint32_t (&w)[kRows][4]) {
  const Rows rows = rows_of<W>(chunk, left);
#pragma unroll
  for (int r = 0; r < kRows; ++r) load_words<W, KEEP>(rows, r, threadIdx.x & (kThreads - 1), w[r]);
  return t.any ? load_tail<W>(chunk, t) : 0u;
}

// Stores that another workgroup of the same launch will read: at device scope they go through the L2 to the
// memory side, so that waiting for their acknowledgement (published_before_here) is all the release that is
// needed -- a release fence would write back all that the L2 holds of the launch's other stores.
template <bool SHARED, typename T>
__device__ __forceinline__ void store_word(T* p, T v) {
  if constexpr (SHARED) __hip_atomic_store((TA_GLOBAL T*)(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else *as_global<T>(p) = v;
}
// Every thread: its device-scope stores and atomics so far have been performed.
__device__ __forceinline__ void published_before_here() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Flags of a lane's elements: bit 4 r + i = element i of row r, kTailFlag = the seventeenth.
constexpr uint32_t kTailFlag = 1u << 16;

// The word of a chunk's mask that this lane writes (`word` of the tensor), if any: lane (8 j + r) of a wavefront row r's word j.
__device__ __forceinline__ bool mask_word_of(const TensorDesc& td, int64_t base, int64_t& word) {
  const int tid = threadIdx.x & (kThreads - 1), sub = tid & 7;
  word = ((base + (int64_t)sub * kRowElems) >> 5) + (tid >> 3);
  return sub < kRows && word < ((td.numel + 31) >> 5);
}

// Mask words of a chunk from every lane's flags (mask_word_of).
template <bool SHARED = false>
__device__ __forceinline__ void store_mask_flags(const TensorDesc& td, int64_t base, uint32_t flags, const Tail& tail) {
  static_assert(kRows == 4, "one word per row, chosen by two bits of the lane");
  const int tid = threadIdx.x & (kThreads - 1);
  const int lane = tid & (kWave - 1);
  const int sub = tid & 7;
  if (tail.any) {
    const uint32_t bits = (uint32_t)__ballot((flags & kTailFlag) != 0u) & 7u;
    if ((uint32_t)tid == tail.owner) flags |= bits << (4 * tail.row);
  }
  const uint32_t w0 = gather_mask_word(flags & 15u, lane), w1 = gather_mask_word((flags >> 4) & 15u, lane);
  const uint32_t w2 = gather_mask_word((flags >> 8) & 15u, lane), w3 = gather_mask_word((flags >> 12) & 15u, lane);
  const uint32_t lo = (sub & 1) ? w1 : w0, hi = (sub & 1) ? w3 : w2;
  int64_t word;
  if (mask_word_of(td, base, word)) store_word<SHARED>(td.mask + word, (sub & 2) ? hi : lo);
}

// What a launch that may have to be taken back overwrote of a chunk (k_stats_ema): curvature and mask words.
struct EmaUndo {
  float* h;
  uint32_t* mask;
};
__device__ __forceinline__ EmaUndo ema_undo(float* undo_h, uint32_t* undo_mask, const TensorDesc& td, int64_t base) {
  const int64_t at = (int64_t)td.undo_slot * kUndoUnit + base;
  return EmaUndo{undo_h + at, undo_mask + (at >> 5)};
}

// Candidate storage.  Each tensor owns kCandLists sub-lists of sub_cap entries plus one overflow
// list of cand_cap entries, each with its own counter in its own 128-byte line: appends from
// different chunks and wavefronts go to different counters, because atomics on one hot address
// serialise.  A batch that does not fit its sub-list spills into the overflow list, so nothing
// is lost as long as the tensor lists at most cand_cap keys in total.
__device__ __forceinline__ uint32_t* cand_counter(uint32_t* counters, uint32_t tensor, uint32_t list) {
  return counters + ((size_t)tensor * (kCandLists + 1) + list) * kCandCounterStride;
}

__device__ __forceinline__ void reset_cand_counters(uint32_t* counters, uint32_t tensor) {
  if (threadIdx.x <= kCandLists) *cand_counter(counters, tensor, threadIdx.x) = 0;
}

// Append a wavefront's candidates of one chunk (`flags`: as for the mask words) with one
// atomic per wavefront.  Slots go element by element and lane by lane inside an element, so that the lanes of
// a store write side by side (lane by lane first, a store of 64 keys touched 64 lines).  The sub-list is chosen
// by (chunk, wavefront), so wavefronts running at the same time use different counters; a tensor that lists all
// its keys (at most 8 wavefronts' worth) has a list of full size for each of them and needs no atomic.
// EfficientNet-B0 set, curvature kernel: 19.4 us with both the other way, 16.0 now.
// In two parts, so that something else can be done while the counter's answer is under way.
struct Appending {
  uint32_t total, list, start;
};
__device__ __forceinline__ Appending append_begin(uint32_t flags, uint32_t chunk_index, uint32_t tensor, const TensorDesc& td,
                                                  uint32_t* counters) {
  Appending a{0, 0, 0};
  if (!__any(flags != 0u)) return a;  // uniform over the wavefront
  const int tid = threadIdx.x & (kThreads - 1);
  a.total = wave_sum((uint32_t)__popc(flags));
  a.list = (chunk_index * (kThreads / kWave) + tid / kWave) % kCandLists;
  if ((tid & (kWave - 1)) == 0) {
    if (td.list_all) *cand_counter(counters, tensor, a.list) = a.total;
    else a.start = atomicAdd(cand_counter(counters, tensor, a.list), a.total);
  }
  return a;
}
template <bool SHARED = false>
__device__ __forceinline__ void append_end(const Appending& a, uint32_t flags, const uint32_t (&h)[kRows][4], uint32_t ht,
                                           const Tail& tail, int64_t base, uint32_t tensor, const TensorDesc& td,
                                           Candidate* cands, uint32_t* counters) {
  if (a.total == 0) return;  // uniform over the wavefront
  const int tid = threadIdx.x & (kThreads - 1);
  const int lane = tid & (kWave - 1);
  const uint32_t total = a.total, list = a.list;
  uint32_t start = a.start, fit = total, ostart = 0;
  if (!td.list_all) {
    if (lane == 0) {
      fit = start < td.sub_cap ? min(total, td.sub_cap - start) : 0u;
      if (fit < total) ostart = atomicAdd(cand_counter(counters, tensor, kCandLists), total - fit);
    }
    start = first_lane(start);
    fit = first_lane(fit);
    ostart = first_lane(ostart);
  }
  Candidate* const own = cands + td.cand_offset + (size_t)list * td.sub_cap + start;
  Candidate* const over = cands + td.cand_offset + (size_t)kCandLists * td.sub_cap + ostart;
  uint32_t before = 0;  // candidates of earlier elements
  const auto put = [&](bool mine, uint32_t value, uint32_t idx) {
    const unsigned long long lanes = __ballot(mine);
    if (mine) {
      const uint32_t rank = before + __builtin_amdgcn_mbcnt_hi((uint32_t)(lanes >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)lanes, 0u));
      // one 8-byte store of a Candidate: idx in the low word, key in the high one
      const uint64_t c = (uint64_t)(value & 0x7fffffffu) << 32 | idx;
      if (rank < fit) store_word<SHARED>(reinterpret_cast<uint64_t*>(own + rank), c);
      else if (ostart + (rank - fit) < td.cand_cap) store_word<SHARED>(reinterpret_cast<uint64_t*>(over + (rank - fit)), c);
    }
    before += (uint32_t)__popcll(lanes);
  };
#pragma unroll
  for (int r = 0; r < kRows; ++r)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      put((flags & (1u << (r * 4 + i))) != 0u, h[r][i], (uint32_t)base + r * kRowElems + tid * kVec + i);
  if (tail.any) put((flags & kTailFlag) != 0u, ht, (uint32_t)base + tail.at);
}

// Visit every listed candidate of a tensor.  s_counts holds the kCandLists + 1 clamped counts.
template <int NT, typename F>
__device__ __forceinline__ void for_each_candidate(const TensorDesc& td, const Candidate* cands,
                                                   const uint32_t* s_counts, F f) {
  const uint32_t lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  for (uint32_t list = wave; list <= kCandLists; list += NT / kWave) {
    const uint32_t cnt = s_counts[list];
    const Candidate* p = cands + td.cand_offset + (size_t)list * td.sub_cap;
    for (uint32_t j = lane; j < cnt; j += kWave) f(p[j]);
  }
}

// ---------------------------------------------------------------------------------------------
// Fallback mask pass for tensors whose mask was not settled by the EMA kernel: re-reads |h| and
// writes the bit mask.  Keys above the range are kept, keys below dropped; keys inside it are
// listed and their bits are set afterwards by k_select_finish.  Called from k_update and k_mask_pass; SHARED: from
// k_select_tail, where a workgroup of the same launch resolves the threshold.
// ---------------------------------------------------------------------------------------------
template <bool SHARED = false>
__device__ __forceinline__ void mask_chunk(const TensorDesc& td, int64_t base, uint32_t mode, uint32_t theta,
                                           uint32_t rng_lo, uint32_t rng_hi, uint32_t chunk_index,
                                           uint32_t tensor, Candidate* cands, uint32_t* counters) {
  uint32_t h[kRows][4];
  const int32_t left = chunk_left(base, td.numel);
  const Tail tail = tail_of(left, (uint32_t)threadIdx.x & (kThreads - 1));
  const uint32_t ht = load_chunk<4>(chunk_of<4>(td.curv, base), left, tail, h);
  // one rule for both modes: keys >= keep_lo are kept, keys in [list_lo, keep_lo) are listed; what lies past the
  // end reads as 0, below both bounds, so it is never kept and never listed
  const bool exact = mode == kSelExact;
  const uint32_t keep_lo = max(exact ? theta : rng_hi, 1u);
  const uint32_t list_lo = exact ? keep_lo : min(max(rng_lo, 1u), keep_lo);
  uint32_t kflags = 0, cflags = 0;
#pragma unroll
  for (int r = 0; r < kRows; ++r) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t key = h[r][i] & 0x7fffffffu;
      kflags |= (key >= keep_lo ? 1u : 0u) << (r * 4 + i);
      cflags |= (key >= list_lo ? 1u : 0u) << (r * 4 + i);
    }
  }
  const uint32_t tkey = ht & 0x7fffffffu;
  if (tkey >= keep_lo) kflags |= kTailFlag;
  if (tkey >= list_lo) cflags |= kTailFlag;
  cflags ^= kflags;  // the kept keys are above list_lo too
  store_mask_flags<SHARED>(td, base, kflags, tail);
  append_end<SHARED>(append_begin(cflags, chunk_index, tensor, td, counters), cflags, h, ht, tail, base, tensor, td, cands, counters);
}

}  // namespace triaccel
