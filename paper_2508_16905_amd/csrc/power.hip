// gfx950 kernels of the power iteration for the top-k eigenvalues of each layer's Hessian
// (Sec. 3.2, third equation): u <- H u / ||H u||, lambda ~ u^T H u / u^T u, carried out for k
// vectors at once with the earlier directions projected out in order (deflation).
//
// The caller supplies, per layer, the k current vectors u_j and the products w_j = H u_j.  The
// orthonormal basis that ordered Gram-Schmidt would produce from W = [w_0 .. w_{k-1}] is W R^-1,
// R being the Cholesky factor of the k x k Gram matrix W^T W.  That needs two streaming passes
// instead of k dependent ones:
//   Gram pass    reads U and W once: W^T W, u_j . w_j, u_j . u_j (fp64 sums, fixed order)
//   layer kernel k x k Cholesky, coefficients of R^-1, Rayleigh quotients, residuals (fp64)
//   apply pass   reads W again, writes q_j = sum_{i<=j} coef_ij w_i over u_j
// Both passes are HBM-bound: 8k bytes per element each.
#include "power.h"

#include <hip/hip_runtime.h>

#include <mutex>

#include "device_util.h"

namespace triaccel {

namespace {

__device__ __forceinline__ constexpr int tri(int i, int j) { return j * (j + 1) / 2 + i; }  // i <= j

template <int K, bool FULL, bool KEEP>
__device__ __forceinline__ void gram_chunk(const PowerDesc& pd, int64_t numel, int64_t base, double (&g)[K * (K + 1) / 2],
                                           double (&c)[K], double (&d)[K]) {
  // the products are read again by the apply pass: KEEP leaves them in the caches (figures at kKeepBytes)
  // the 2k loads of R rows are in flight together, and the accumulators leave room for several wavefronts per SIMD to
  // overlap their loads with the fp64 arithmetic (one row, and R: 1000 chunks, k = 1 24.1 and 20.0 us an iteration, k = 2
  // 32.5 and 30.4; 400 chunks, k = 1 12.5 and 11.7; 6000 chunks, k = 3 202 and 190, k = 4 the same)
  const auto add = [&](const uint32_t (&ub)[K], const uint32_t (&wb)[K]) {
#pragma unroll
    for (int j = 0; j < K; ++j) {
      const double wj = (double)u2f(wb[j]), uj = (double)u2f(ub[j]);
      c[j] = fma(uj, wj, c[j]);
      d[j] = fma(uj, uj, d[j]);
#pragma unroll
      for (int i = 0; i <= j; ++i) g[tri(i, j)] = fma((double)u2f(wb[i]), wj, g[tri(i, j)]);
    }
  };
  constexpr int R = K <= 2 ? 4 : K <= 4 ? 2 : 1;
  static_assert(kRows % R == 0, "whole steps");
#pragma unroll 1
  for (int r0 = 0; r0 < kRows; r0 += R) {
    if (!FULL && chunk_left(base + (int64_t)r0 * kRowElems, numel) <= 0) break;
    uint32_t u[R][K][4], w[R][K][4];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int64_t at = base + (int64_t)(r0 + r) * kRowElems;
      const int32_t left = FULL ? kRowElems : chunk_left(at, numel);
#pragma unroll
      for (int j = 0; j < K; ++j) {
        load_row4<FULL>(pd.u + at + (int64_t)j * pd.stride, threadIdx.x, left, u[r][j]);
        load_row4<FULL, KEEP>(pd.hu + at + (int64_t)j * pd.stride, threadIdx.x, left, w[r][j]);
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        uint32_t ub[K], wb[K];
#pragma unroll
        for (int j = 0; j < K; ++j) {
          ub[j] = u[r][j][e];
          wb[j] = w[r][j][e];
        }
        add(ub, wb);
        // one element's conversions to double at a time: those of all four took 80 registers more
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  if constexpr (!FULL) {
    const float* const up = pd.u + base;
    const float* const wp = pd.hu + base;
    const Tail tail = tail_of(chunk_left(base, numel), threadIdx.x);
    if (tail.any) {
      uint32_t ub[K], wb[K];
#pragma unroll
      for (int j = 0; j < K; ++j) {
        ub[j] = load_tail<4>(up + (int64_t)j * pd.stride, tail);
        wb[j] = load_tail<4>(wp + (int64_t)j * pd.stride, tail);
      }
      add(ub, wb);
    }
  }
}

// Gram pass: one workgroup per segment (`seg` consecutive chunks of one tensor).  The pointers come with the
// kernel's arguments when the call has few enough tensors, and the first segment of a tensor leaves them in the
// table for the apply pass: a copy from host memory ahead of the pass cost the stream 10 us a call.
// Bound by HBM: 447 MB (11.2 M parameters, k = 5) in 70 us, 6.3 TB/s; with 2 wavefronts per SIMD (206 registers),
// segments of 8 chunks and reductions through LDS it took 79.
template <int K, bool KEEP>
__global__ __launch_bounds__(kThreads, K <= 5 ? 3 : 1) void k_power_gram(const TensorDesc* __restrict__ tds,
                                                                         PowerDescArg arg, PowerDesc* __restrict__ pds,
                                                                         const SegRef* __restrict__ segs, uint32_t seg,
                                                                         double* __restrict__ partials) {
  constexpr int NG = K * (K + 1) / 2, PP = NG + 2 * K;
  const SegRef sr = segs[blockIdx.x];
  const int64_t numel = tds[sr.tensor].numel;
  const uint32_t n_chunks = tds[sr.tensor].n_chunks;
  const PowerDesc pd = arg.count ? arg.e[sr.tensor] : pds[sr.tensor];
  if (arg.count && sr.index == 0 && threadIdx.x == 0) pds[sr.tensor] = pd;
  double g[NG], c[K], d[K];
#pragma unroll
  for (int i = 0; i < NG; ++i) g[i] = 0.0;
#pragma unroll
  for (int j = 0; j < K; ++j) c[j] = d[j] = 0.0;
  const uint32_t c0 = sr.index * seg;
  const uint32_t c1 = min(c0 + seg, n_chunks);
  // the ragged chunk, if it is this segment's, comes after the loop over the full ones: with both bodies in one
  // loop the sums were held twice (206 registers at k = 5, 2 wavefronts per SIMD)
  const uint32_t full = min(c1, (uint32_t)(numel / kChunk));
  for (uint32_t ch = c0; ch < full; ++ch) gram_chunk<K, true, KEEP>(pd, numel, (int64_t)ch * kChunk, g, c, d);
  if (full < c1) gram_chunk<K, false, KEEP>(pd, numel, (int64_t)full * kChunk, g, c, d);
  // lanes, then wavefronts, in a fixed order
  __shared__ double s_part[kThreads / kWave][PP];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
#pragma unroll
  for (int i = 0; i < NG; ++i) {
    const double v = wave_sum_f64(g[i]);
    if (lane == 0) s_part[wave][i] = v;
  }
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const double vc = wave_sum_f64(c[j]), vd = wave_sum_f64(d[j]);
    if (lane == 0) {
      s_part[wave][NG + j] = vc;
      s_part[wave][NG + K + j] = vd;
    }
  }
  __syncthreads();
  if (threadIdx.x < PP) {
    const int e = threadIdx.x;
    partials[(size_t)blockIdx.x * PP + e] = ((s_part[0][e] + s_part[1][e]) + s_part[2][e]) + s_part[3][e];
  }
}

// Value of lane `src` (fp64), every lane its own `src`.
__device__ __forceinline__ double from_lane(double v, int src) {
  const int lo = __builtin_amdgcn_ds_bpermute(src * 4, __double2loint(v)), hi = __builtin_amdgcn_ds_bpermute(src * 4, __double2hiint(v));
  return __hiloint2double(hi, lo);
}

// Per-layer kernel: one workgroup per tensor adds the segment partials (fixed order) and its first wavefront
// factorises the k x k Gram matrix, one entry per lane.  A vector whose remainder after projecting out the earlier
// directions is numerically nothing (pivot <= 1e-12 of its own squared norm) gets a zero column.
// Bound by chains of fp64 divisions and square roots of some 200 cycles each: a column at a time by one thread there were
// 55 of them one after the other at k = 5 and 110 at k = 8, here 4 and a few for each of the k steps.  ResNet-18 set,
// k = 5: the call 147.2 -> 145.1 us; 3 M parameters, k = 8: 84.2 -> 78.8; 11 tensors of 60 elements, k = 8: 22.6 -> 16.9.
// (Sixteen wavefronts for the sums: a tensor of 144 segments 9 of them each, in one or two batches of loads.)
constexpr int kLayerThreads = 1024;
template <int K>
__global__ __launch_bounds__(kLayerThreads) void k_power_layer(const TensorDesc* __restrict__ tds,
                                                          const uint32_t* __restrict__ seg_first,
                                                          uint32_t seg, const double* __restrict__ partials,
                                                          PowerLayer* state, LayerDev* layers, int latch) {
  constexpr int NG = K * (K + 1) / 2, PP = NG + 2 * K, N = kMaxPowerK;
  static_assert(PP <= kWave && N * N == kWave, "one lane per partial entry, one per matrix entry");
  const uint32_t l = blockIdx.x;
  const uint32_t n_segs = (tds[l].n_chunks + seg - 1) / seg;
  const double* p = partials + (size_t)seg_first[l] * PP;
  const int e = threadIdx.x & (kWave - 1), part = threadIdx.x / kWave;
  double acc = 0.0;
  if (e < PP)
#pragma unroll 8
    for (uint32_t s = part; s < n_segs; s += kLayerThreads / kWave) acc += p[(size_t)s * PP + e];
  __shared__ double s_acc[kLayerThreads / kWave][kWave];
  s_acc[part][e] = acc;
  __syncthreads();
  if (part != 0) return;
  double sum = 0.0;
#pragma unroll
  for (int q = 0; q < kLayerThreads / kWave; ++q) sum += s_acc[q][e];
  const auto total = [&](int t) { return from_lane(sum, t); };
  PowerLayer& st = state[l];
  // quotients, residuals ||w - lambda u|| / ||u|| and norms from the sums (zero iterate: both 0): lane j, vector j
  {
    const int j = e < K ? e : 0;
    const double gjj = total(tri(j, j)), c = total(NG + j), d = total(NG + K + j);
    double lam = 0.0, res = 0.0;
    if (d > 0.0) {
      lam = c / d;
      const double r2 = gjj - 2.0 * lam * c + lam * lam * d;
      res = sqrt(r2 > 0.0 ? r2 : 0.0) / sqrt(d);
    }
    if (e < N) {
      st.rayleigh[e] = e < K ? (float)lam : 0.0f;
      st.resid[e] = e < K ? (float)res : 0.0f;
      st.hnorm[e] = e < K ? (float)sqrt(gjj) : 0.0f;
    }
    double lam_max = 0.0;
#pragma unroll
    for (int q = 0; q < K; ++q) lam_max = fmax(lam_max, fabs(from_lane(lam, q)));
    if (e == 0) {
      st.lambda_max = (float)lam_max;
      if (latch) layers[l].lambda_power = (float)lam_max;
    }
  }
  // lane N i + j, i <= j: entry (i, j) of the Gram matrix G, of its Cholesky factor R (G = R^T R) and of R^-1 = T; in the
  // products the order of the subtractions is that of the left-looking forms
  const int i = e / N, j = e % N;
  const bool in = i <= j && j < K;
  const double gram = total(in ? tri(i, j) : 0);
  const double g = in ? gram : 0.0;
  double s = g, r = 0.0;      // s: G_ij less the products of the rows above
  double diag[K];             // R_pp, the same in all lanes
  uint32_t deficient = 0;
#pragma unroll
  for (int q = 0; q < K; ++q) {
    const double piv = from_lane(s, q * N + q), full = from_lane(g, q * N + q);
    const bool def = piv <= 1e-12 * full;
    diag[q] = def ? 0.0 : sqrt(piv);
    if (def) deficient |= 1u << q;
    const double row = def ? 0.0 : s / diag[q];  // R_qj in the lanes of row q
    if (i == q) r = j == q ? diag[q] : row;
    const double a = from_lane(r, q * N + i), b = from_lane(r, q * N + j);
    if (i > q) s -= a * b;
  }
  // q_j = (w_j - sum_{p<j} R_pj q_p) / R_jj in terms of the w_i
  double t = i == j ? 1.0 : 0.0;
#pragma unroll
  for (int q = 0; q < K; ++q) {
    const double done = ((deficient >> q) & 1u) ? 0.0 : t / diag[q];
    if (j == q) t = done;
    const double a = from_lane(t, i * N + q), b = from_lane(r, q * N + j);
    if (i <= q && q < j) t -= a * b;
  }
  st.coef[i][j] = in ? t : 0.0;
  if (e == 0) st.deficient = deficient;
}

template <int K, bool FULL>
__device__ __forceinline__ void apply_chunk(const PowerDesc& pd, int64_t numel, int64_t base,
                                            const double (&t)[K * (K + 1) / 2]) {
#pragma unroll
  for (int r = 0; r < kRows; ++r) {
    const int64_t at = base + (int64_t)r * kRowElems;
    const int32_t left = FULL ? kRowElems : chunk_left(at, numel);
    if (!FULL && left <= 0) break;
    const float* const wp = pd.hu + at;
    uint32_t w[K][4];
#pragma unroll
    for (int j = 0; j < K; ++j) load_row4<FULL>(wp + (int64_t)j * pd.stride, threadIdx.x, left, w[j]);
#pragma unroll
    for (int j = 0; j < K; ++j) {
      uint32_t q[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        double acc = 0.0;
#pragma unroll
        for (int i = 0; i <= j; ++i) acc = fma(t[tri(i, j)], (double)u2f(w[i][e]), acc);
        q[e] = f2u((float)acc);
      }
      store_row4<FULL>(pd.u + at + (int64_t)j * pd.stride, threadIdx.x, left, q);
    }
    if constexpr (!FULL) {
      const Tail tail = tail_of(left, threadIdx.x);
      if (tail.any && left < kRowElems) {
        double wt[K];
#pragma unroll
        for (int j = 0; j < K; ++j) wt[j] = (double)u2f(load_tail<4>(wp + (int64_t)j * pd.stride, tail));
#pragma unroll
        for (int j = 0; j < K; ++j) {
          double acc = 0.0;
#pragma unroll
          for (int i = 0; i <= j; ++i) acc = fma(t[tri(i, j)], wt[i], acc);
          store_tail<kFP32>(pd.u + at + (int64_t)j * pd.stride, tail, f2u((float)acc));
        }
      }
    }
  }
}

// Apply pass: one workgroup per chunk.
template <int K>
__global__ __launch_bounds__(kThreads) void k_power_apply(const TensorDesc* __restrict__ tds,
                                                          const PowerDesc* __restrict__ pds,
                                                          const ChunkRef* __restrict__ chunks,
                                                          const PowerLayer* __restrict__ state) {
  constexpr int NG = K * (K + 1) / 2;
  const ChunkRef cr = chunks[blockIdx.x];
  const int64_t numel = tds[cr.tensor].numel;
  const PowerDesc pd = pds[cr.tensor];
  double t[NG];
#pragma unroll
  for (int j = 0; j < K; ++j)
#pragma unroll
    for (int i = 0; i <= j; ++i) t[tri(i, j)] = state[cr.tensor].coef[i][j];
  const int64_t base = (int64_t)cr.index * kChunk;
  if (base + kChunk <= numel) apply_chunk<K, true>(pd, numel, base, t);
  else apply_chunk<K, false>(pd, numel, base, t);
}

// Part of the pointer table of a call with many tensors.
__global__ __launch_bounds__(kPowerArgTensors) void k_power_descs(PowerDescArg a, PowerDesc* __restrict__ pds) {
  if (threadIdx.x < a.count) pds[threadIdx.x] = a.e[threadIdx.x];
}

template <int K>
hipError_t launch_k(const PowerTables& t, const PowerDesc* descs, int latch, hipStream_t s, hipEvent_t* ev) {
  hipError_t e;
  PowerDescArg arg{};
  if (descs) {
    for (uint32_t first = 0; first < t.n_tensors; first += kPowerArgTensors) {
      arg.count = t.n_tensors - first < (uint32_t)kPowerArgTensors ? t.n_tensors - first : (uint32_t)kPowerArgTensors;
      for (uint32_t i = 0; i < arg.count; ++i) arg.e[i] = descs[first + i];
      if (t.n_tensors <= (uint32_t)kPowerArgTensors) break;
      hipLaunchKernelGGL(k_power_descs, dim3(1), dim3(kPowerArgTensors), 0, s, arg, t.descs + first);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (t.n_tensors > (uint32_t)kPowerArgTensors) arg.count = 0;
  }
  if (ev && (e = hipEventRecord(ev[0], s)) != hipSuccess) return e;
  // total_chunks * kChunk: the vectors' length to within a chunk per tensor
  const bool keep = (uint64_t)t.total_chunks * kChunk * K * 4 <= kKeepBytes;
  const auto gram = keep ? k_power_gram<K, true> : k_power_gram<K, false>;
  hipLaunchKernelGGL(gram, dim3(t.total_segs), dim3(kThreads), 0, s, t.tensors, arg, t.descs, t.segs,
                     t.seg, t.partials);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (ev && (e = hipEventRecord(ev[1], s)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_power_layer<K>, dim3(t.n_tensors), dim3(kLayerThreads), 0, s, t.tensors, t.seg_first, t.seg,
                     t.partials, t.state, t.layers, latch);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (ev && (e = hipEventRecord(ev[2], s)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_power_apply<K>, dim3(t.total_chunks), dim3(kThreads), 0, s, t.tensors, t.descs, t.chunks,
                     t.state);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (ev && (e = hipEventRecord(ev[3], s)) != hipSuccess) return e;
  return hipSuccess;
}

// ---------------------------------------------------------------------------------------------
// The iteration for callers that cannot allocate: every table and partial sum the kernels above
// use lives in one fixed device array.  Host code never uses the array's name as an address: the
// device address is looked up once per GPU (each GPU holds its own copy) and passed to the kernels.
// ---------------------------------------------------------------------------------------------
constexpr size_t align256(size_t b) { return (b + 255) & ~size_t(255); }
constexpr size_t kStaticMaxSegs = kStaticMaxChunks / 8 + kStaticMaxTensors;
static_assert(power_seg(16383, 8) == 4 && power_seg(kStaticMaxChunks, 8) == 8 && kStaticMaxChunks / 8 >= 16384 / 4 &&
                  power_seg(1201, 1) == 4,
              "segments of any set fit the array");
constexpr size_t kOffTensors = 0;
constexpr size_t kOffDescs = kOffTensors + align256(sizeof(TensorDesc) * kStaticMaxTensors);
constexpr size_t kOffSegFirst = kOffDescs + align256(sizeof(PowerDesc) * kStaticMaxTensors);
constexpr size_t kOffChunks = kOffSegFirst + align256(sizeof(uint32_t) * kStaticMaxTensors);
constexpr size_t kOffSegs = kOffChunks + align256(sizeof(ChunkRef) * kStaticMaxChunks);
constexpr size_t kOffPartials = kOffSegs + align256(sizeof(SegRef) * kStaticMaxSegs);
constexpr size_t kOffState = kOffPartials + align256(sizeof(double) * power_partial_len(kMaxPowerK) * kStaticMaxSegs);
constexpr size_t kScratchBytes = kOffState + align256(sizeof(PowerLayer) * kStaticMaxTensors);
static_assert(kScratchBytes < (size_t(5) << 20), "the fixed array is meant to stay a few MiB");

static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
unsigned char* g_scratch_ptr[kMaxDevices] = {};  // device address of `scratch` on each GPU (null: not looked up yet)
std::mutex g_scratch_mutex;

struct StaticEntry {
  float* u;
  const float* hu;
  int64_t stride;
  int64_t numel;
  uint32_t first_chunk;
  uint32_t first_seg;
};
struct StaticBatchArg {
  uint32_t first;  // index of the batch's first tensor
  uint32_t count;
  StaticEntry e[kStaticBatch];
};
static_assert(sizeof(StaticBatchArg) <= 3072, "passed by value as a kernel argument");

// Table kernel: workgroup b writes the tables of tensor first + b (descriptor, chunk and segment lists).
__global__ __launch_bounds__(kThreads) void k_static_tables(StaticBatchArg a, uint32_t seg, unsigned char* base) {
  const StaticEntry en = a.e[blockIdx.x];
  const uint32_t l = a.first + blockIdx.x;
  const uint32_t nc = (uint32_t)((en.numel + kChunk - 1) / kChunk);
  const uint32_t ns = (nc + seg - 1) / seg;
  if (threadIdx.x == 0) {
    TensorDesc td{};
    td.numel = en.numel;
    td.first_chunk = en.first_chunk;
    td.n_chunks = nc;
    reinterpret_cast<TensorDesc*>(base + kOffTensors)[l] = td;
    reinterpret_cast<PowerDesc*>(base + kOffDescs)[l] = PowerDesc{en.u, en.hu, en.stride};
    reinterpret_cast<uint32_t*>(base + kOffSegFirst)[l] = en.first_seg;
  }
  ChunkRef* chunks = reinterpret_cast<ChunkRef*>(base + kOffChunks) + en.first_chunk;
  for (uint32_t c = threadIdx.x; c < nc; c += kThreads) chunks[c] = ChunkRef{l, c};
  SegRef* segs = reinterpret_cast<SegRef*>(base + kOffSegs) + en.first_seg;
  for (uint32_t q = threadIdx.x; q < ns; q += kThreads) segs[q] = SegRef{l, q};
}

__global__ void k_static_export(const PowerLayer* __restrict__ state, PowerInfoOut* __restrict__ out, int n) {
  const int l = blockIdx.x * blockDim.x + threadIdx.x;
  if (l >= n) return;
  PowerInfoOut o;
  for (int j = 0; j < kMaxPowerK; ++j) {
    o.rayleigh[j] = state[l].rayleigh[j];
    o.resid[j] = state[l].resid[j];
    o.hnorm[j] = state[l].hnorm[j];
  }
  o.deficient = state[l].deficient;
  o.lambda_max = state[l].lambda_max;
  o.lambda_latched = 0.0f;
  out[l] = o;
}

}  // namespace

hipError_t power_static_prepare() {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[dev]) return hipSuccess;
  void* p = nullptr;
  e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess) return e;
  if (!p) return hipErrorInvalidSymbol;
  g_scratch_ptr[dev] = static_cast<unsigned char*>(p);
  return hipSuccess;
}

hipError_t launch_power_iter_static(const StaticTensor* tensors, int n, int k, PowerInfoOut* info, hipStream_t s) {
  hipError_t e = power_static_prepare();
  if (e != hipSuccess) return e;
  int dev = -1;
  if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
  unsigned char* base = g_scratch_ptr[dev];
  if (n == 0) return hipSuccess;
  // tables: the prefix sums are formed here, the lists are written on the device
  uint32_t chunk_pos = 0, seg_pos = 0, total = 0;
  for (int i = 0; i < n; ++i) total += (uint32_t)((tensors[i].numel + kChunk - 1) / kChunk);
  const uint32_t seg = power_seg(total, k);
  for (int first = 0; first < n; first += kStaticBatch) {
    StaticBatchArg a{};
    a.first = (uint32_t)first;
    a.count = (uint32_t)(n - first < kStaticBatch ? n - first : kStaticBatch);
    for (uint32_t i = 0; i < a.count; ++i) {
      const StaticTensor& t = tensors[first + (int)i];
      const uint32_t nc = (uint32_t)((t.numel + kChunk - 1) / kChunk);
      a.e[i] = StaticEntry{t.u, t.hu, t.stride, t.numel, chunk_pos, seg_pos};
      chunk_pos += nc;
      seg_pos += (nc + seg - 1) / seg;
    }
    hipLaunchKernelGGL(k_static_tables, dim3(a.count), dim3(kThreads), 0, s, a, seg, base);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  PowerTables t{};
  t.tensors = reinterpret_cast<const TensorDesc*>(base + kOffTensors);
  t.chunks = reinterpret_cast<const ChunkRef*>(base + kOffChunks);
  t.layers = nullptr;  // only written when a value is latched into an optimizer handle: never here
  t.descs = reinterpret_cast<PowerDesc*>(base + kOffDescs);
  t.segs = reinterpret_cast<SegRef*>(base + kOffSegs);
  t.seg_first = reinterpret_cast<uint32_t*>(base + kOffSegFirst);
  t.partials = reinterpret_cast<double*>(base + kOffPartials);
  t.state = reinterpret_cast<PowerLayer*>(base + kOffState);
  t.n_tensors = (uint32_t)n;
  t.total_chunks = chunk_pos;
  t.total_segs = seg_pos;
  t.seg = seg;
  // every partial sum and every record the kernels read is written earlier in this same call, so
  // nothing in the array has to start at zero
  if ((e = launch_power_iter(t, nullptr, k, 0, s, nullptr)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_static_export, dim3((n + kWave - 1) / kWave), dim3(kWave), 0, s, t.state, info, n);
  return hipGetLastError();
}

hipError_t launch_power_iter(const PowerTables& t, const PowerDesc* descs, int k, int latch, hipStream_t s, hipEvent_t* ev) {
  switch (k) {
    case 1: return launch_k<1>(t, descs, latch, s, ev);
    case 2: return launch_k<2>(t, descs, latch, s, ev);
    case 3: return launch_k<3>(t, descs, latch, s, ev);
    case 4: return launch_k<4>(t, descs, latch, s, ev);
    case 5: return launch_k<5>(t, descs, latch, s, ev);
    case 6: return launch_k<6>(t, descs, latch, s, ev);
    case 7: return launch_k<7>(t, descs, latch, s, ev);
    case 8: return launch_k<8>(t, descs, latch, s, ev);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace triaccel
