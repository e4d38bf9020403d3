// Power iteration for the top-k eigenvalues of each layer's Hessian (Sec. 3.2, third equation):
// device tables and host-callable launchers (defined in power.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "common.h"

namespace triaccel {

constexpr int kMaxPowerK = 8;  // vectors per layer the workspace can be sized for
// Chunks of one tensor that one workgroup of the Gram pass sums, for k vectors.  One, while segments of 4 would give a
// compute unit hardly more than one workgroup: the rows of a segment follow one after the other.  Above that 4, and 8
// from 16,384 chunks, as more partial sums to add per tensor cost more than the shorter segments gain.  The line is
// where a set of one tensor, which has the most to add, gains nothing more.  With 7 and 8 vectors 512 workgroups fit
// the chip (two wavefronts per SIMD; 768 and more with fewer vectors), and 700 to 900 of them leave a second round
// nearly empty: 3 to 4 % lost, so the line is below that.
// An iteration on 20 tensors, us, with segments of 4 and of 1 chunks:
//   chunks   k = 1            k = 3            k = 5            k = 6            k = 8
//   500      16.8 and 13.5    28.1 and 20.6    43.4 and 35.9    50.0 and 41.3    62.4 and 54.2
//   640      17.1 and 14.3    32.3 and 26.2    48.3 and 43.5    56.1 and 52.4    71.9 and 71.7
//   760      18.4 and 15.4    34.7 and 30.3    52.5 and 49.7    60.2 and 58.6    78.7 and 81.1
//   900      19.7 and 16.2    39.4 and 36.6    60.7 and 58.0    68.8 and 68.1    91.1 and 93.4
//   1200     22.8 and 17.6    51.6 and 45.7    80.2 and 72.1    95.3 and 88.8    126 and 115
//   1500     25.1 and 22.1    57.7 and 55.1    91.0 and 87.0    108 and 103      142 and 140
//   2800     39.0 and 36.1    94.4 and 95.8    150 and 151      181 and 181      257 and 248
// One tensor of 1200 chunks: 23.0 and 22.3, 51.2 and 47.7, 75.9 and 73.8, 90.3 and 86.1, 120 and 112; of 1500: 26.1 and 25.9,
// 55.9 and 58.8, 87.3 and 89.6, 103 and 105, 136 and 138; of 2800: 40.8 and 49.7, 93.8 and 105, 149 and 160, 178 and 188,
// 239 and 248.  (Segments of 2 lie between the two.)
// k is the call's, in both entry points: the order of the sums, and with it the last bits of the result, is the same
// with a handle of any size and without one.  A handle keeps the tables of both kinds of k if they differ.
constexpr int kPowerFewK = 6;
constexpr uint32_t power_seg(uint32_t total_chunks, int k) {
  return total_chunks <= (k <= kPowerFewK ? 1200u : 640u) ? 1u : total_chunks < 16384 ? 4u : 8u;
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
