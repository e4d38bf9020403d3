// Order in which the chunks of a tensor are rewritten when its storage size changes in place
// (2 <-> 4 bytes per element), as plain functions that the kernels, their launcher and a host-side
// replay of the schedule all use.
//
// Element range [lo, hi) occupies bytes [s lo, s hi) at element size s.  NARROWING (4 -> 2): chunk c
// writes into bytes that held the old data of chunk c / 2 (its parent), so a chunk may be stored once
// its parent has been loaded.  WIDENING (2 -> 4): chunk c writes over the old data of chunks 2c and
// 2c + 1 (its children), so a chunk may be stored once both children have been loaded.  Chunk 0 is
// its own parent / child: its loads must precede its own stores.
//
// The dependence is a binary tree, and the subtrees rooted at the chunks [A, 2A) are independent of
// each other: level v of the subtree of root r is the contiguous run of chunks [r 2^v, (r + 1) 2^v),
// its stores land on the old bytes of level v - 1 (narrowing) or v + 1 (widening) of the same
// subtree, and never on the old bytes of its own level.  One workgroup walks one subtree, level by
// level with a workgroup barrier between levels (root to leaves when narrowing, leaves to root when
// widening) and without waiting for any other workgroup.  What a root itself depends on lies in
// [A / 2, A) (narrowing) -- chunks done by an earlier launch.  A step therefore needs
//   stage 0      chunks [0, top)
//   stage j >= 1 chunks [root_j, root_j 2^depth_j): root_j workgroups per tensor, depth_j levels each
// with root_1 = top and root_{j+1} = root_j 2^depth_j, in this order for a narrowing tensor and in
// the reverse order for a widening one.
//
// Stage 0 has two forms.  In a set without a subtree stage it is one workgroup per tensor that takes the
// chunks one after the other, with a barrier in every chunk: no launch of its own is needed.  With subtree
// stages, `top` workgroups compute one chunk each in launch 0 and put the new values into a scratch area of
// the tensor's own; they are copied into place by resize_copy_launch, after all chunks that hold old data
// there (those below 2 top) have been loaded by earlier launches: no chain, at the price of moving 2 or 4
// bytes per element of `top` chunks twice.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#define TA_HD __host__ __device__ inline
#else
#define TA_HD inline
#endif

namespace triaccel {

constexpr uint32_t kResizeMaxStages = 8;     // stage 0 plus up to 7 subtree stages
constexpr uint32_t kResizeTop = 16;          // chunks of stage 0 when subtree stages follow, large sets
constexpr uint32_t kResizeTopSmall = 64;     // the same, sets below kResizeBigSet: fewer levels in all, so fewer
                                             // stages and shallower subtrees
// Up to 256 of them where that pays.  More chunks side by side make the subtrees shallower and more, and give launch 0
// of a narrowing tensor, which takes 27 us for the first 64 chunks of 12 tensors, more to do; they cost their copy, so they are at
// most a quarter of the longest tensor, or all but one in short sets, whose launches have room.  Every tensor is offered as many work
// items as the longest, so their number is limited too, by the chunks there are: a ragged set of 60 tensors (40 M) took
// 354 us instead of 230 without that.  Tensors of more than 4096 chunks have two subtree stages and more roots from their
// first: one of some 9000 chunks among 8 of 60 M 240 and 257.  A step in which every tensor is resized, us, with 64 and with this many: 12
// of 1024 chunks 214 and 193 (256), 15 264 and 239, 4 89 and 72, one of 1000 39 and 25, 8 of 500 79 and 74, 4 of 160 22.8 and
// 21.7 (128), 6 ragged of 6 M 44 and 36; with 128 all the same 30 of 200 118 and 125, 30 of 300 189 and 195.  512 of 1024: 75
// instead of 72 for 4, 24.1 instead of 24.6 for one.  With step sizes per element 12 of 1024 254 and 220, one of 1000 50 and 30,
// 6 ragged of 6 M 59 and 48, 60 ragged of 40 M (64 either way) 324 and 324.
// The rule ends at 1024 chunks, the longest tensor of the local form, with which it was made; nothing in the scheme ends there.  From
// 1025 to 4096 chunks, still one subtree stage, 256 would gain as well: 12 of 1025 220 and 200, one of 1025 40 and 26, 4 of 1500
// 134 and 104, 8 of 2000 289 and 238, 3 of 4096 259 and 182, one of 4096 130 and 69, 12 ragged of 25 M 170 and 122; 30 ragged of 30 M
// 160 and 162, steps without a change the same within 1 %.
constexpr uint32_t kResizeTopMax = 256;
constexpr uint32_t kResizeShortSet = 4096;   // chunks in the whole set
constexpr uint32_t kResizeOneSubtree = 1024; // longest tensor of the sets that the rule is for
constexpr uint32_t kResizeTopOnly = 128;     // tensors up to this many chunks: stage 0 alone
constexpr uint32_t kResizeBigSet = 16384;    // chunks in the whole set from which a launch more costs nothing
                                             // (= kLaunchBoundChunks of the step's other kernels)

struct ResizePlan {
  uint32_t n_stages;                  // 1 + number of subtree stages
  uint32_t top;                       // chunks [0, top) belong to stage 0
  uint32_t root[kResizeMaxStages];    // stage j >= 1: roots [root[j], 2 root[j])
  uint32_t depth[kResizeMaxStages];   // stage j >= 1: levels 0 .. depth[j] - 1
};

// Plan for a set of `n_tensors` whose largest tensor has `max_chunks` chunks.  Small sets are bound by the number of
// launches, so they get deep subtrees (up to 6 levels, 63 chunks per workgroup) and as few stages as
// possible; large sets get shallow ones (up to 4 levels, 15 chunks) for parallelism inside a tensor.
TA_HD ResizePlan make_resize_plan(uint32_t max_chunks, uint32_t total_chunks, uint32_t n_tensors) {
  ResizePlan p{};
  p.n_stages = 1;
  if (max_chunks <= kResizeTopOnly) {
    p.top = max_chunks ? max_chunks : 1u;
    return p;
  }
  p.top = total_chunks >= kResizeBigSet ? kResizeTop : kResizeTopSmall;
  if (total_chunks < kResizeBigSet && max_chunks <= kResizeOneSubtree) {
    const uint32_t most = total_chunks <= kResizeShortSet ? max_chunks - 1 : max_chunks / 4;
    const uint32_t chunks = total_chunks + total_chunks / 8, items = chunks > kResizeShortSet ? chunks : kResizeShortSet;
    // work items of a launch: as many roots as chunks of stage 0
    while (2 * p.top <= most && 2 * p.top <= kResizeTopMax && (uint64_t)n_tensors * 2 * (2 * p.top) <= items) p.top *= 2;
  }
  uint32_t levels = 0;  // smallest count with top << levels >= max_chunks
  while (((uint64_t)p.top << levels) < max_chunks) ++levels;
  const uint32_t dmax = total_chunks >= kResizeBigSet ? 4u : 6u;
  const uint32_t n_sub = (levels + dmax - 1) / dmax;
  const uint32_t base = levels / n_sub, rem = levels % n_sub;
  uint32_t root = p.top;
  for (uint32_t j = 1; j <= n_sub; ++j) {
    p.root[j] = root;
    p.depth[j] = base + (j > n_sub - rem ? 1u : 0u);  // the later (wider) stages take the deeper trees
    root <<= p.depth[j];
  }
  p.n_stages = 1 + n_sub;
  return p;
}

// Stage that launch `launch` (0 .. n_stages - 1) performs for a tensor.
TA_HD uint32_t resize_stage_of_launch(const ResizePlan& p, uint32_t launch, bool narrowing) {
  return narrowing ? launch : p.n_stages - 1u - launch;
}

// Launch in which a scratch copy of chunks [0, top) is put into place (plans with subtree stages): a
// narrowing chunk overwrites old data of [0, top) only, a widening one of [0, 2 top), whose last part is
// loaded by stage 1.
TA_HD uint32_t resize_copy_launch(const ResizePlan& p, bool narrowing) { return narrowing ? 1u : p.n_stages - 1u; }

// Workgroups one tensor needs in a stage (stage 0 in one workgroup: one).
TA_HD uint32_t resize_stage_roots(const ResizePlan& p, uint32_t stage) { return stage == 0 ? 1u : p.root[stage]; }

// Stage 0 in one workgroup: chunks [0, min(top, n_chunks)), ascending when narrowing, descending when widening.
// `chunk_op(c)` must load the chunk, pass a workgroup barrier, then store it.
template <class ChunkOp>
TA_HD void resize_walk_top(const ResizePlan& p, uint32_t n_chunks, bool narrowing, ChunkOp&& chunk_op) {
  const uint32_t n = n_chunks < p.top ? n_chunks : p.top;
  for (uint32_t i = 0; i < n; ++i) chunk_op(narrowing ? i : n - 1u - i);
}

// Order of workgroups for a launch that has one for every chunk of the set and in which chunk 0's workgroup does
// that walk: every tensor's chunk 0, then the others.  The walks start first and lie side by side in the grid, so
// all compute units get some; in the tensors' own order those of tensors of 8, 16, 24, ... chunks all fell to one
// of the chip's eight dies, to which workgroups go in turn.  Steps in which every tensor is resized, own order and
// heads first: 500 tensors of 16 chunks 634 and 116 us, 60 of 96 898 and 204, 100 of 128 1935 and 300, 300 of 21
// 142 and 109, EfficientNet-B0 set 176 and 176 (its ordinary step 20.4 and 20.0).
// `put(tensor, chunk)` appends an entry; n_chunks(t) is the number of chunks of tensor t.
template <class Chunks, class Put>
inline void heads_first(uint32_t n_tensors, Chunks&& n_chunks, Put&& put) {
  for (uint32_t t = 0; t < n_tensors; ++t) put(t, 0u);
  for (uint32_t t = 0; t < n_tensors; ++t)
    for (uint32_t c = 1; c < n_chunks(t); ++c) put(t, c);
}

// Stage j >= 1, workgroup `r` (0 <= r < root[j]) of a tensor: the subtree of chunk root[j] + r.
// `chunk_op(c)` loads and stores one chunk (its loads and stores never overlap: c >= 1);
// `level_done()` is the workgroup barrier between two levels.
template <class ChunkOp, class LevelDone>
TA_HD void resize_walk_subtree(const ResizePlan& p, uint32_t stage, uint32_t r, uint32_t n_chunks, bool narrowing,
                               ChunkOp&& chunk_op, LevelDone&& level_done) {
  const uint32_t first = p.root[stage] + r, depth = p.depth[stage];
  for (uint32_t i = 0; i < depth; ++i) {
    const uint32_t v = narrowing ? i : depth - 1u - i;
    const uint64_t lo = (uint64_t)first << v;
    if (lo >= n_chunks) {
      if (narrowing) break;  // deeper levels lie further out still
      continue;
    }
    const uint64_t end = lo + ((uint64_t)1 << v);
    const uint32_t hi = end < n_chunks ? (uint32_t)end : n_chunks;
    for (uint32_t c = (uint32_t)lo; c < hi; ++c) chunk_op(c);
    level_done();
  }
}

}  // namespace triaccel
