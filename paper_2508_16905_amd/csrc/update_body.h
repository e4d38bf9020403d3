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
// One function, update_as, loads, computes and stores a chunk; a kernel that rewrites a tensor in place at
// another element size has it put one workgroup barrier between the loads and the stores, at a single place
// that every thread passes (BARRIER).
// ELEM: the step size is scaled per element instead of per layer (Sec. 3.2, "Step size scaling",
// applied to each entry of the sparsified curvature): eta_i = lr / fma(alpha, a_i, 1) with
// a_i = |h_i| if the entry is in the mask (|h_i| >= theta and |h_i| > 0), else 0; reads h once more.
// ---------------------------------------------------------------------------------------------
struct StepSize {
  float neg_eta;       // per-layer form: -eta_l
  float lr, alpha;     // element-wise form
  uint32_t theta_key;  // element-wise form: bit pattern of the mask threshold
};

// A lane's 16 elements of one chunk: gradient and parameters as they lie in memory (fp32: 4 words a row, 16 bits: 2)
// until update_math widens them in place, and the momentum; then the new values.
struct ChunkRegs {
  uint32_t th[kRows][4];
  uint32_t m[kRows][4];
  uint32_t g[kRows][4];
};
struct CurvRegs {
  uint32_t h[kRows][4];
};

// The chunk's arrays: gradient, parameters, momentum and curvature from its first element on.
struct ChunkArrays {
  const void* g;
  const void* th;
  const void* m;
  const void* h;
  int32_t left;
};
template <int GW, int PW>
__device__ __forceinline__ ChunkArrays chunk_arrays(const TensorDesc& td, int64_t base) {
  return ChunkArrays{chunk_of<GW>(td.grad, base), chunk_of<PW>(static_cast<const void*>(td.param), base),
                     chunk_of<4>(static_cast<const void*>(td.mom), base), chunk_of<4>(static_cast<const void*>(td.curv), base),
                     chunk_left(base, td.numel)};
}

template <int GW, int PW, bool MOM, bool ELEM>
__device__ __forceinline__ void update_fetch(const ChunkArrays& a, uint32_t tid, ChunkRegs& r, CurvRegs& c) {
  // Row by row, the arrays interleaved; the compiler pairs the rows of an array.  (Measured over 48 placements of the
  // arrays in memory each, with accesses at plain addresses: issuing the loads array by array instead is 2 % slower
  // on average, rotating the row order between the arrays changes nothing.  Holding the compiler to the written order
  // through the descriptors: no difference that the placements let show.)
  const Rows grows = rows_of<GW>(a.g, a.left), trows = rows_of<PW>(a.th, a.left), mrows = rows_of<4>(a.m, a.left);
  const Rows hrows = rows_of<4>(a.h, a.left);
#pragma unroll
  for (int q = 0; q < kRows; ++q) {
    load_words<GW>(grows, q, tid, r.g[q]);
    load_words<PW>(trows, q, tid, r.th[q]);
    if constexpr (MOM) load_words<4>(mrows, q, tid, r.m[q]);
    if constexpr (ELEM) load_words<4>(hrows, q, tid, c.h[q]);
  }
}

// A lane's seventeenth element (Tail).
struct TailRegs {
  uint32_t g, th, m, h;
};
template <int GW, int PW, bool MOM, bool ELEM>
__device__ __forceinline__ TailRegs update_fetch_tail(const ChunkArrays& a, const Tail& t) {
  TailRegs r{0, 0, 0, 0};
  if (t.any) {
    r.g = load_tail<GW>(a.g, t);
    r.th = load_tail<PW>(a.th, t);
    if constexpr (MOM) r.m = load_tail<4>(a.m, t);
    if constexpr (ELEM) r.h = load_tail<4>(a.h, t);
  }
  return r;
}

// One element, fp32 bit patterns: new momentum and parameter in place.
template <bool MOM, bool ELEM>
__device__ __forceinline__ void update_element(float inv_scale, float wd, float mu, const StepSize& ss, uint32_t g, uint32_t& th,
                                               uint32_t& m, uint32_t h) {
  const float gt = u2f(g) * inv_scale;
  const float d = fmaf(wd, u2f(th), gt);
  const float mm = MOM ? fmaf(mu, u2f(m), d) : d;
  m = f2u(mm);
  float neg_eta = ss.neg_eta;
  if constexpr (ELEM) {
    const uint32_t key = h & 0x7fffffffu;
    const float a = (key >= ss.theta_key && key != 0u) ? u2f(key) : 0.0f;
    const float den = fmaf(ss.alpha, a, 1.0f);
    neg_eta = -(ss.lr / den);
  }
  th = f2u(fmaf(neg_eta, mm, u2f(th)));
}

template <int GD, int PD, bool MOM, bool ELEM>
__device__ __forceinline__ void update_math(float inv_scale, float wd, float mu, const StepSize& ss, ChunkRegs& r,
                                            const CurvRegs& c) {
#pragma unroll
  for (int q = 0; q < kRows; ++q) {
    widen4<GD>(r.g[q]);
    widen4<PD>(r.th[q]);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      update_element<MOM, ELEM>(inv_scale, wd, mu, ss, r.g[q][i], r.th[q][i], r.m[q][i], ELEM ? c.h[q][i] : 0u);
  }
}

// The same for the seventeenth element, and its stores.
template <int GD, int PD, bool MOM, bool ELEM>
__device__ __forceinline__ void update_tail(int nd, float inv_scale, float wd, float mu, const StepSize& ss,
                                            const Tail& t, TailRegs r, void* th, void* m) {
  r.g = widen1<GD>(r.g);
  r.th = widen1<PD>(r.th);
  update_element<MOM, ELEM>(inv_scale, wd, mu, ss, r.g, r.th, r.m, r.h);
  if (nd == kFP32) store_tail<kFP32>(th, t, r.th);
  else if (nd == kBF16) store_tail<kBF16>(th, t, r.th);
  else store_tail<kFP16>(th, t, r.th);
  if constexpr (MOM) store_tail<kFP32>(m, t, r.m);
}

// `th`, `m`: the chunk's parameters and momentum from its first element on.
template <int ND, bool MOM>
__device__ __forceinline__ void update_store(void* th, void* m, int32_t left, uint32_t tid, ChunkRegs& r) {
  constexpr int W = kWords<ND>;
  const Rows trows = rows_of<W>(th, left), mrows = rows_of<4>(m, left);
#pragma unroll
  for (int q = 0; q < kRows; ++q) {
    narrow4<ND>(r.th[q]);
    store_words<W>(trows, q, tid, r.th[q]);
    if constexpr (MOM) store_words<4>(mrows, q, tid, r.m[q]);
  }
}

// One chunk: loads, `decide` while they are under way (false: leave without a store), arithmetic, stores.  Gradient, old
// and new precision are uniform over a workgroup: it branches once into a body specialised for the first two, and in
// that for the stores.  Whether there is a momentum buffer is uniform over the
// set and a parameter of the kernel: as a branch inside the body it made the compiler fetch the first
// row of a chunk ahead of the branch and wait for it there, two memory latencies per chunk instead of
// one (50 M parameters that all change size: 252 -> 236 us a step; 11.2 M ordinary: 55.2 -> 54.6 us).
// BARRIER: a workgroup barrier between loads and stores.  `to`: where the parameters go (the tensor's start).
template <bool ELEM, bool MOM, bool BARRIER, int GD, int PD, typename Decide>
__device__ __forceinline__ bool update_as(const TensorDesc& td, const int& nd, int64_t base, float inv_scale, float wd, float mu,
                                          const StepSize& ss, uint32_t tid, Decide&& decide, void* to) {
  constexpr int GW = kWords<GD>, PW = kWords<PD>;
  const ChunkArrays a = chunk_arrays<GW, PW>(td, base);
  ChunkRegs r;
  CurvRegs c;
  update_fetch<GW, PW, MOM, ELEM>(a, tid, r, c);
  const Tail tail = tail_of(a.left, tid);
  const TailRegs rt = update_fetch_tail<GW, PW, MOM, ELEM>(a, tail);
  if (!decide()) return false;
  update_math<GD, PD, MOM, ELEM>(inv_scale, wd, mu, ss, r, c);
  if constexpr (BARRIER) __syncthreads();
  void* const m = chunk_of<4>(static_cast<void*>(td.mom), base);
  switch (nd) {
    case kFP32: update_store<kFP32, MOM>(chunk_of<4>(to, base), m, a.left, tid, r); break;
    case kBF16: update_store<kBF16, MOM>(chunk_of<2>(to, base), m, a.left, tid, r); break;
    default: update_store<kFP16, MOM>(chunk_of<2>(to, base), m, a.left, tid, r); break;
  }
  if (tail.any)
    update_tail<GD, PD, MOM, ELEM>(nd, inv_scale, wd, mu, ss, tail, rt, nd == kFP32 ? chunk_of<4>(to, base) : chunk_of<2>(to, base),
                                   m);
  return true;
}

template <bool ELEM, bool MOM, bool BARRIER, int GD, typename Decide>
__device__ __forceinline__ bool update_from(const TensorDesc& td, int pd, const int& nd, int64_t base, float inv_scale, float wd,
                                            float mu, const StepSize& ss, uint32_t tid, Decide&& decide, void* to) {
  switch (pd) {
    case kFP32: return update_as<ELEM, MOM, BARRIER, GD, kFP32>(td, nd, base, inv_scale, wd, mu, ss, tid, decide, to);
    case kBF16: return update_as<ELEM, MOM, BARRIER, GD, kBF16>(td, nd, base, inv_scale, wd, mu, ss, tid, decide, to);
    default: return update_as<ELEM, MOM, BARRIER, GD, kFP16>(td, nd, base, inv_scale, wd, mu, ss, tid, decide, to);
  }
}

template <bool ELEM, bool MOM, bool BARRIER = false, typename Decide>
__device__ __forceinline__ bool update_any(const TensorDesc& td, int pd, const int& nd, int64_t base, float inv_scale, float wd,
                                           float mu, const StepSize& ss, uint32_t tid, Decide&& decide, void* to) {
  switch (td.grad_dtype) {
    case kFP32: return update_from<ELEM, MOM, BARRIER, kFP32>(td, pd, nd, base, inv_scale, wd, mu, ss, tid, decide, to);
    case kBF16: return update_from<ELEM, MOM, BARRIER, kBF16>(td, pd, nd, base, inv_scale, wd, mu, ss, tid, decide, to);
    default: return update_from<ELEM, MOM, BARRIER, kFP16>(td, pd, nd, base, inv_scale, wd, mu, ss, tid, decide, to);
  }
}

template <bool ELEM, bool MOM, bool BARRIER = false, typename Decide>
__device__ __forceinline__ bool update_any(const TensorDesc& td, int pd, const int& nd, int64_t base, float inv_scale, float wd,
                                           float mu, const StepSize& ss, uint32_t tid, Decide&& decide) {
  return update_any<ELEM, MOM, BARRIER>(td, pd, nd, base, inv_scale, wd, mu, ss, tid, decide, td.param);
}

}  // namespace triaccel
