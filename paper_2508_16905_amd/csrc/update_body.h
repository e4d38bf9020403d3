// Body of the fused update + cast, shared by the kernels that apply it in place (update.hip) and
// stage by stage while the storage size changes (update_resize.hip).
#pragma once
#include "device_util.h"

namespace triaccel {

// ---------------------------------------------------------------------------------------------
// Stage 5: fused update + cast.  Per element, fp32:
//   theta = widen(param);  gt = widen(g) * inv_scale;  d = fma(wd, theta, gt);
//   m = fma(mu, m, d) (m = d without a buffer);  theta' = fma(-eta, m, theta);
//   store theta' in the layer's new precision, round to nearest even.
// The body comes in two halves -- load + arithmetic into registers, then the stores -- so that a
// kernel that rewrites a tensor in place at another element size can put its one workgroup barrier
// between them, at a single place that every thread passes.
// ELEM: the step size is scaled per element instead of per layer (Sec. 3.2, "Step size scaling",
// applied to each entry of the sparsified curvature): eta_i = lr / fma(alpha, a_i, 1) with
// a_i = |h_i| if the entry is in the mask (|h_i| >= theta and |h_i| > 0), else 0; reads h once more.
// ---------------------------------------------------------------------------------------------
struct StepSize {
  float neg_eta;       // per-layer form: -eta_l
  float lr, alpha;     // element-wise form
  uint32_t theta_key;  // element-wise form: bit pattern of the mask threshold
};

// A lane's 16 elements of one chunk: parameters, momentum and gradient as loaded, then the new values.
struct ChunkRegs {
  float th[kRows][4];
  float m[kRows][4];
  float g[kRows][4];
};
struct CurvRegs {
  float h[kRows][4];
};

template <int GD, int PD, bool FULL, bool MOM, bool ELEM>
__device__ __forceinline__ void update_fetch(const TensorDesc& td, int64_t base, int tid, ChunkRegs& r, CurvRegs& c) {
  // Row by row, the arrays interleaved.  (Measured over 48 placements of the arrays in memory each,
  // with the accesses in the global address space: issuing the loads array by array instead is 2 %
  // slower on average, rotating the row order between the arrays changes nothing.)
#pragma unroll
  for (int q = 0; q < kRows; ++q) {
    const int64_t idx = base + q * kRowElems + tid * kVec;
    if constexpr (FULL) {
      load4<GD>(td.grad, idx, r.g[q]);
      load4<PD>(td.param, idx, r.th[q]);
      if constexpr (MOM) load4<kFP32>(td.mom, idx, r.m[q]);
      if constexpr (ELEM) load4<kFP32>(td.curv, idx, c.h[q]);
    } else {
      load4_guard<GD>(td.grad, idx, td.numel, 0.0f, r.g[q]);
      load4_guard<PD>(td.param, idx, td.numel, 0.0f, r.th[q]);
      if constexpr (MOM) load4_guard<kFP32>(td.mom, idx, td.numel, 0.0f, r.m[q]);
      if constexpr (ELEM) load4_guard<kFP32>(td.curv, idx, td.numel, 0.0f, c.h[q]);
    }
  }
}

template <bool MOM, bool ELEM>
__device__ __forceinline__ void update_math(float inv_scale, float wd, float mu, const StepSize& ss, ChunkRegs& r,
                                            const CurvRegs& c) {
#pragma unroll
  for (int q = 0; q < kRows; ++q) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float gt = r.g[q][i] * inv_scale;
      const float d = fmaf(wd, r.th[q][i], gt);
      const float mm = MOM ? fmaf(mu, r.m[q][i], d) : d;
      r.m[q][i] = mm;
      float neg_eta = ss.neg_eta;
      if constexpr (ELEM) {
        const uint32_t key = f2u(c.h[q][i]) & 0x7fffffffu;
        const float a = (key >= ss.theta_key && key != 0u) ? u2f(key) : 0.0f;
        const float den = fmaf(ss.alpha, a, 1.0f);
        neg_eta = -(ss.lr / den);
      }
      r.th[q][i] = fmaf(neg_eta, mm, r.th[q][i]);
    }
  }
}

template <int ND, bool FULL, bool MOM>
__device__ __forceinline__ void update_store(const TensorDesc& td, int64_t base, int tid, const ChunkRegs& r) {
#pragma unroll
  for (int q = 0; q < kRows; ++q) {
    const int64_t idx = base + q * kRowElems + tid * kVec;
    if constexpr (FULL) {
      store4<ND>(td.param, idx, r.th[q]);
      if constexpr (MOM) store4<kFP32>(td.mom, idx, r.m[q]);
    } else {
      store4_guard<ND>(td.param, idx, td.numel, r.th[q]);
      if constexpr (MOM) store4_guard<kFP32>(td.mom, idx, td.numel, r.m[q]);
    }
  }
}

// Gradient, old and new precision are uniform over a workgroup: each half branches once per chunk
// into a body specialised for its combination.  Whether there is a momentum buffer is uniform over the
// set and a parameter of the kernel: as a branch inside the body it made the compiler fetch the first
// row of a chunk ahead of the branch and wait for it there, two memory latencies per chunk instead of
// one (50 M parameters that all change size: 252 -> 236 us a step; 11.2 M ordinary: 55.2 -> 54.6 us).
template <bool ELEM, bool MOM, int GD, int PD>
__device__ __forceinline__ void update_fetch2(const TensorDesc& td, int64_t base, int tid, ChunkRegs& r, CurvRegs& c) {
  if (base + kChunk <= td.numel) update_fetch<GD, PD, true, MOM, ELEM>(td, base, tid, r, c);
  else update_fetch<GD, PD, false, MOM, ELEM>(td, base, tid, r, c);
}

template <bool ELEM, bool MOM, int GD>
__device__ __forceinline__ void update_fetch1(int pd, const TensorDesc& td, int64_t base, int tid, ChunkRegs& r, CurvRegs& c) {
  switch (pd) {
    case kFP32: update_fetch2<ELEM, MOM, GD, kFP32>(td, base, tid, r, c); break;
    case kBF16: update_fetch2<ELEM, MOM, GD, kBF16>(td, base, tid, r, c); break;
    default: update_fetch2<ELEM, MOM, GD, kFP16>(td, base, tid, r, c); break;
  }
}

template <bool ELEM, bool MOM>
__device__ __forceinline__ void update_fetch_any(const TensorDesc& td, int pd, int64_t base, int tid, ChunkRegs& r,
                                                 CurvRegs& c) {
  switch (td.grad_dtype) {
    case kFP32: update_fetch1<ELEM, MOM, kFP32>(pd, td, base, tid, r, c); break;
    case kBF16: update_fetch1<ELEM, MOM, kBF16>(pd, td, base, tid, r, c); break;
    default: update_fetch1<ELEM, MOM, kFP16>(pd, td, base, tid, r, c); break;
  }
}

template <bool ELEM, bool MOM>
__device__ __forceinline__ void update_load_any(const TensorDesc& td, int pd, int64_t base, float inv_scale, float wd,
                                                float mu, const StepSize& ss, int tid, ChunkRegs& r) {
  CurvRegs c;
  update_fetch_any<ELEM, MOM>(td, pd, base, tid, r, c);
  update_math<MOM, ELEM>(inv_scale, wd, mu, ss, r, c);
}

template <bool MOM, int ND>
__device__ __forceinline__ void update_store1(const TensorDesc& td, int64_t base, int tid, const ChunkRegs& r) {
  if (base + kChunk <= td.numel) update_store<ND, true, MOM>(td, base, tid, r);
  else update_store<ND, false, MOM>(td, base, tid, r);
}

template <bool MOM>
__device__ __forceinline__ void update_store_any(const TensorDesc& td, int nd, int64_t base, int tid,
                                                 const ChunkRegs& r) {
  switch (nd) {
    case kFP32: update_store1<MOM, kFP32>(td, base, tid, r); break;
    case kBF16: update_store1<MOM, kBF16>(td, base, tid, r); break;
    default: update_store1<MOM, kFP16>(td, base, tid, r); break;
  }
}

// One chunk, loads then stores, for the kernels in which they cannot overlap.
template <bool ELEM, bool MOM>
__device__ __forceinline__ void update_any(const TensorDesc& td, int pd, int nd, int64_t base, float inv_scale,
                                           float wd, float mu, const StepSize& ss, int tid) {
  ChunkRegs r;
  update_load_any<ELEM, MOM>(td, pd, base, inv_scale, wd, mu, ss, tid, r);
  update_store_any<MOM>(td, nd, base, tid, r);
}

}  // namespace triaccel
