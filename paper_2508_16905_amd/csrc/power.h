// Power iteration for the top-k eigenvalues of each layer's Hessian (Sec. 3.2, third equation):
// device tables and host-callable launchers (defined in power.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "common.h"

namespace triaccel {

constexpr int kMaxPowerK = 8;  // vectors per layer the workspace can be sized for
// Chunks of one tensor that one workgroup of the Gram pass sums, for k vectors.  Sets that fit the chip with a workgroup
// for every chunk (768 at k = 5) get one: the rows of a segment follow one after the other.  Above that segments of 4,
// and of 8 from 16,384 chunks, where more partial sums to add per tensor cost more than the shorter segments gain.
// An iteration, us, with segments of 1 and 4 chunks: 200 chunks, k = 1 12.6 and 18.6, k = 5 20.8 and 34.6, k = 8 30.4
// and 49.1; 400: 13.8 and 19.9, 31.1 and 41.5, 50.9 and 60.5; 600: 15.3 and 22.0, 44.3 and 48.0, 72.3 and 70.8; 768:
// 17.3 and 22.9, 51.9 and 53.9, 82.1 and 80.8; 1000: 19.8 and 24.5, 66.1 and 63.7, 101 and 96; 2700: 42.9 and 36.6,
// 153 and 146, 246 and 244 (segments of 2 lie between the two).
// k is the call's, in both entry points: the order of the sums, and with it the last bits of the result, is the same
// with a handle of any size and without one.  A handle keeps the tables of both kinds of k if they differ.
constexpr int kPowerFewK = 5;
constexpr uint32_t power_seg(uint32_t total_chunks, int k) {
  return total_chunks <= (k <= kPowerFewK ? 768u : 512u) ? 1u : total_chunks < 16384 ? 4u : 8u;
}

// Doubles one workgroup of the Gram pass leaves for k vectors: the upper triangle of W^T W
// (W = [H u_0 .. H u_{k-1}]), then u_j . (H u_j), then u_j . u_j.
constexpr int power_partial_len(int k) { return k * (k + 1) / 2 + 2 * k; }

// Per tensor: the k vectors of one call.  Vector j occupies elements [j * stride, j * stride + numel).
struct PowerDesc {
  float* u;
  const float* hu;
  int64_t stride;
};

struct SegRef {
  uint32_t tensor;
  uint32_t index;  // segment number inside the tensor: chunks [index * seg, (index + 1) * seg)
};

// Pointers of a call with few enough tensors, passed by value to its first kernel.
constexpr int kPowerArgTensors = 128;
struct PowerDescArg {
  uint32_t count;  // 0: read the table
  PowerDesc e[kPowerArgTensors];
};
static_assert(sizeof(PowerDescArg) <= 3200, "passed by value as a kernel argument");
// Up to this many tensors the pointers travel that way, kPowerArgTensors a launch; for more the launches cost as much
// as a copy from pinned memory, which is what such calls make unless the stream is being captured.  An iteration of
// tensors of 3000 elements, k = 2, arguments (its two speeds) and copy: 129 tensors 15.8 / 19.4 and 18.3 us, 256
// 16.4 / 19.5 and 17.9, 384 20 / 24 and 19.6, 640 28 / 33 and 23.7, 1000 38 / 45 and 42, 2000 72 / 81 and 61, 4000
// 133 / 148 and 94.
constexpr uint32_t kPowerArgMax = 2 * kPowerArgTensors;

// Per-tensor result of the last call.
struct PowerLayer {
  // q_j = sum_{i <= j} coef[i][j] * (H u_i): the orthonormalisation in terms of the supplied vectors
  double coef[kMaxPowerK][kMaxPowerK];
  float rayleigh[kMaxPowerK];
  float resid[kMaxPowerK];
  float hnorm[kMaxPowerK];
  uint32_t deficient;
  float lambda_max;  // max_j |rayleigh_j| of this call
};

struct PowerTables {
  const TensorDesc* tensors;  // numel and chunk counts (shared with the optimizer step)
  const ChunkRef* chunks;
  LayerDev* layers;
  PowerDesc* descs;
  SegRef* segs;
  uint32_t* seg_first;  // per tensor: index of its first segment
  double* partials;     // total_segs x power_partial_len(k)
  PowerLayer* state;
  uint32_t n_tensors;
  uint32_t total_chunks;
  uint32_t total_segs;
  uint32_t seg;  // power_seg
};

// One iteration on k vectors per tensor: Gram pass, per-layer factorisation, apply pass.  With
// `ev` (four events) the boundaries of the three kernels are recorded on the stream.  `descs` (host, n_tensors
// entries) travels as kernel arguments; null: the table t.descs is filled already, or is by a copy enqueued before.
hipError_t launch_power_iter(const PowerTables& t, const PowerDesc* descs, int k, int latch, hipStream_t s, hipEvent_t* ev);

// The same iteration without a handle and without any allocation: tables and partial sums live in a
// fixed device array of this library (one per GPU), rebuilt by a small kernel on every call.
constexpr int kStaticMaxTensors = 256;      // tensors per call
constexpr int kStaticMaxChunks = 65536;     // sum over the tensors of ceil(numel / kChunk): 268,435,456 elements
constexpr int kStaticBatch = 64;            // tensor descriptions handed to the table kernel per launch

struct StaticTensor {
  float* u;
  const float* hu;
  int64_t stride;
  int64_t numel;
};

// Exported per-tensor record (layout of triaccel_power_info).
struct PowerInfoOut {
  float rayleigh[kMaxPowerK];
  float resid[kMaxPowerK];
  float hnorm[kMaxPowerK];
  uint32_t deficient;
  float lambda_max;
  float lambda_latched;
};

// Looks up (once per device) the address of the fixed array on the current device.
hipError_t power_static_prepare();
// `tensors` is a host array of n entries; `info` a device array of n records.  The caller has checked
// the limits above.  Calls on one GPU share the array: they must not overlap in time.
hipError_t launch_power_iter_static(const StaticTensor* tensors, int n, int k, PowerInfoOut* info, hipStream_t s);

}  // namespace triaccel
