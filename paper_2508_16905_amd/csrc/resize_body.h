// Work of one launch of the in-place resize (tensors whose storage size changes between 2 and 4
// bytes per element), as a device function: the first launch rides in the grid of the update kernel,
// the later ones are launches of their own (update_resize.hip).
#pragma once
#include "resize_schedule.h"
#include "update_body.h"

namespace triaccel {

// The tensors are rewritten in place in the order resize_schedule.h lays down: stage 0 (the first chunks of
// a tensor), then subtree stages in which every workgroup walks the levels of its own subtree of chunks with
// a barrier between levels.  No workgroup waits for another; what a stage depends on was done by an
// earlier launch.  Launch q performs stage q for the narrowing tensors of the step's list and stage
// n_stages - 1 - q for the widening ones; the slots [0, top) of a tensor belong to stage 0, the others to the
// subtrees.
//
// With one workgroup taking the 16 first chunks one after the other, as the form without subtree stages still
// does, that stage is a chain of 2-6 us per chunk; side by side the first 64 chunks of 12 tensors took 26 us with
// the rest of that launch (they are up to 256 now, kResizeTopMax).
// Scratch of the tensor for chunk c < top: kChunk elements of 4 bytes.
__device__ __forceinline__ char* resize_scratch(const TensorDesc& td, char* scratch, uint32_t c) {
  return scratch + ((size_t)td.resize_slot + c) * (kChunk * 4);
}

// Copies the new values of chunk c from the scratch area into place.
template <int THREADS>
__device__ __forceinline__ void resize_copy(const TensorDesc& td, const char* src, uint32_t esz, uint32_t c) {
  const int64_t base = (int64_t)c * kChunk, left = td.numel - base;
  const uint32_t bytes = (uint32_t)(left < kChunk ? left : kChunk) * esz;
  char* const dst = static_cast<char*>(td.param) + base * esz;
  for (uint32_t off = threadIdx.x * 16; off < bytes; off += THREADS * 16) {
    if (off + 16 <= bytes) {
      *as_global<v4f>(dst + off) = *as_global<v4f>(src + off);
    } else {
      for (uint32_t b = off; b < bytes; b += 2) *as_global<uint16_t>(dst + b) = *as_global<uint16_t>(src + b);
    }
  }
}

// One tensor's work of slot `r` in launch `launch`.  Uniform over the workgroup (it contains barriers), which
// consists of GROUPS times kThreads threads that take the chunks of a level in turn (launch 0: GROUPS = 1).
template <bool ELEM, bool MOM, int GROUPS = 1>
__device__ __forceinline__ void resize_item(const TensorDesc& desc, int old_code, int new_code, const StepSize& ss,
                                            const StepTables& tab, uint32_t launch, uint32_t slot,
                                            const StepScalars& sc) {
  const ResizePlan& plan = tab.plan;
  char* const scratch = tab.resize_scratch;
  const float wd = tab.hyper.weight_decay, mu = tab.hyper.momentum;
  // The same in every lane, but the compiler does not see it here: without saying so every access through a buffer
  // descriptor becomes a loop over the descriptors that the lanes might hold (128 chunks one after the other: 211 us
  // with plain addresses, 248 with such loops).
  TensorDesc td = desc;
  td.param = uniform(desc.param);
  td.grad = uniform(desc.grad);
  td.mom = uniform(desc.mom);
  td.curv = uniform(desc.curv);
  td.numel = (int64_t)uniform((uint32_t)desc.numel);  // below 2^31
  td.n_chunks = uniform(desc.n_chunks);
  td.grad_dtype = (int32_t)uniform((uint32_t)desc.grad_dtype);
  td.resize_slot = uniform(desc.resize_slot);
  const int pd = (int)uniform((uint32_t)old_code), nd = (int)uniform((uint32_t)new_code);
  const uint32_t r = uniform(slot);
  const uint32_t tid = threadIdx.x & (kThreads - 1);
  const uint32_t group = uniform(threadIdx.x / kThreads);
  const bool narrowing = elem_size(nd) < elem_size(pd);
  if (plan.n_stages == 1) {
    if (r != 0 || launch != 0) return;
    resize_walk_top(plan, td.n_chunks, narrowing, [&](uint32_t c) {
      // chunk 0 overwrites itself; a later chunk overwrites what an earlier one loaded
      update_any<ELEM, MOM, true>(td, pd, nd, (int64_t)c * kChunk, sc.inv_scale, wd, mu, ss, tid, [] { return true; });
    });
    return;
  }
  const uint32_t stage = resize_stage_of_launch(plan, launch, narrowing);
  // in place for the subtrees, into the scratch area for a chunk of stage 0
  void* to = td.param;
  uint32_t sub = r - plan.top;
  if (r < plan.top) {
    if (r >= td.n_chunks) return;
    if (launch != 0) {
      if (launch == resize_copy_launch(plan, narrowing)) resize_copy<GROUPS * kThreads>(td, resize_scratch(td, scratch, r), elem_size(nd), r);
      return;
    }
    to = resize_scratch(td, scratch, r) - (int64_t)r * kChunk * elem_size(nd);
  } else {
    if (stage == 0 || sub >= resize_stage_roots(plan, stage) || plan.root[stage] + sub >= td.n_chunks) return;
  }
  const auto chunk = [&](uint32_t c) {
    if (GROUPS > 1 && c % GROUPS != group) return;
    update_any<ELEM, MOM>(td, pd, nd, (int64_t)c * kChunk, sc.inv_scale, wd, mu, ss, tid, [] { return true; }, to);
  };
  // a chunk of stage 0 is a walk of one level and one chunk
  if (r < plan.top) chunk(r);
  else resize_walk_subtree(plan, stage, sub, td.n_chunks, narrowing, chunk, [&]() { __syncthreads(); });
}

// Work items of a launch are (list entry, slot) pairs of the `count` tensors on the list, `slots` per entry (enough for either direction);
// workgroup `wg` of `n_wg` takes the items wg,
// wg + n_wg, ...  The list and its length are written on the device by the kernel that takes the layers'
// decisions, so the work is offered on every step and nothing happens when the list is empty.
template <bool ELEM, bool MOM, int GROUPS = 1>
__device__ __forceinline__ void resize_items(const StepTables& tab, const TensorDesc* __restrict__ tds, uint32_t count,
                                             uint32_t launch, uint32_t slots, uint32_t wg, uint32_t n_wg, const StepScalars& sc) {
  const uint32_t* list = tab.trans_list + (sc.step_id & 1u) * tab.n_tensors;
  const uint64_t items = (uint64_t)count * slots;
  for (uint64_t item = wg; item < items; item += n_wg) {
    const uint32_t l = uniform(list[item / slots]);
    const uint32_t r = (uint32_t)(item % slots);
    const LayerDev& ls = tab.layers[l];
    const StepSize ss{-ls.eta, sc.lr, tab.hyper.alpha, ls.theta_key};
    const TensorDesc td = tds[l];
    resize_item<ELEM, MOM, GROUPS>(td, ls.prev_code, ls.code, ss, tab, launch, r, sc);
  }
}

// Work items per list entry and workgroups offered to launch `launch`.
struct ResizeGrid {
  uint32_t slots;
  uint32_t grid;
};
inline ResizeGrid resize_grid(const ResizePlan& plan, uint32_t launch, uint32_t n_tensors, bool small) {
  uint32_t slots = 1;
  if (plan.n_stages > 1) {
    // a narrowing tensor is at stage `launch`, a widening one at the mirrored stage
    const uint32_t sa = launch, sb = plan.n_stages - 1u - launch;
    const uint32_t a = sa ? resize_stage_roots(plan, sa) : 0u, b = sb ? resize_stage_roots(plan, sb) : 0u;
    slots = plan.top + (a > b ? a : b);
  }
  uint64_t grid = (uint64_t)n_tensors * slots;
  // the workgroups are offered on every step: small sets loop over their items rather than pay for more
  const uint64_t cap = small ? 1024u : 65536u;
  if (grid > cap) grid = cap;
  return ResizeGrid{slots, (uint32_t)grid};
}

}  // namespace triaccel
