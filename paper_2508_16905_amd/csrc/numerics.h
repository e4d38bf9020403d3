// Device-side number-format conversions and 4-element vector accessors (gfx950).
//
// IEEE round-to-nearest-even, overflow to infinity, subnormals produced exactly, NaN kept NaN.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace triaccel {

enum : int { kFP16 = 0, kBF16 = 1, kFP32 = 2 };

__device__ __forceinline__ uint32_t f2u(float f) { return __float_as_uint(f); }
__device__ __forceinline__ float u2f(uint32_t u) { return __uint_as_float(u); }

// Conversions use the gfx950 conversion instructions through the language casts: v_cvt_f16_f32 /
// v_cvt_pk_bf16_f32 round to nearest even (the mode HIP kernels run in), overflow to infinity
// and produce subnormals exactly; v_cvt_f32_f16 and the 16-bit shift of bfloat16 are exact.
// The result is checked against the CPU oracle for all 2^32 inputs by the GPU test suite.
//
// The fp32 value is pinned in a register before it is narrowed: otherwise the compiler may merge
// the producing fused multiply-add with the conversion into one mixed-precision instruction that
// rounds the exact product-sum once, straight to 16 bits, instead of first to fp32 and then to 16
// bits as the update is defined.
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float x) {
  asm volatile("" : "+v"(x));
  const __bf16 b = (__bf16)x;
  return (uint32_t)__builtin_bit_cast(unsigned short, b);
}

__device__ __forceinline__ uint32_t f32_to_f16_bits(float x) {
  asm volatile("" : "+v"(x));
  const _Float16 h = (_Float16)x;
  return (uint32_t)__builtin_bit_cast(unsigned short, h);
}

__device__ __forceinline__ float f16_bits_to_f32(uint32_t h) {
  return (float)__builtin_bit_cast(_Float16, (unsigned short)h);
}

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t b) { return u2f(b << 16); }

// ---- 4 consecutive elements, index multiple of 4, base 16-byte aligned ------------------------
// Every tensor is streamed exactly once per kernel, so the vector accesses carry the
// non-temporal hint (measured on MI355X: read-only streaming 6.5 -> 7.3 TB/s, read-modify-write
// 5.3 -> 5.7 TB/s), except loads of an array that a later kernel of the same step reads again (KEEP): the
// hint also keeps the data out of the caches.
typedef float v4f __attribute__((ext_vector_type(4)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));

// Tensor pointers reach the kernels through tables in memory, so the compiler cannot tell that they
// point to global memory and would emit FLAT accesses.  A wavefront cannot count flat loads back
// one by one (they may be served by another memory), so it waits for ALL its outstanding loads
// before it uses the first result -- in the middle of a batch of loads that serialises their
// latencies.  Every tensor is device (global) memory by the library's contract: say so.
#define TA_GLOBAL __attribute__((address_space(1)))

template <typename T>
__device__ __forceinline__ const TA_GLOBAL T* as_global(const void* p) {
  return (const TA_GLOBAL T*)(p);
}
template <typename T>
__device__ __forceinline__ TA_GLOBAL T* as_global(void* p) {
  return (TA_GLOBAL T*)(p);
}

// Four elements as they lie in memory: 4 words in fp32, the first 2 words in 16 bits.  W: that number, which is also
// the bytes of an element.  They are widened where they are used (widen4), so that nothing waits for a load before
// all loads of a chunk are under way, and 16-bit data takes half the registers until then.
template <int DT>
constexpr int kWords = DT == kFP32 ? 4 : 2;

// The rows of a chunk are accessed through a buffer descriptor of its whole fours: the hardware reads what lies past
// them as 0 and drops stores there, so a ragged chunk goes the same straight way as a full one (a lane's four
// elements are inside or outside as a whole).  The last left % 4 elements are a seventeenth element of lanes 0 .. 2 of
// the wavefront they belong to (Tail).  With guarded accesses lane by lane, each behind a branch, the chunk with a
// tensor's end took 0.7 us longer than a full one in the statistics and 2.3 us in the update: the last workgroup of
// every small tensor (EfficientNet-B0 set, 213 tensors, 16-bit storage: 18.3 -> 16.8 us a step; 41 ragged tensors of
// 9.7 M, Fisher source: 64.7 -> 59.7; two-layer perceptron with a probe: 37.0 -> 35.0).
typedef __amdgpu_buffer_rsrc_t Rows;
constexpr int kRowLanes = 256;     // lanes of a row, 4 elements each
constexpr int kBufferRaw = 0x00020000;  // descriptor word 3: untyped 32-bit accesses, offsets in bytes
constexpr int kNonTemporal = 2;    // cache-policy bit of the buffer instructions

// `chunk`: its first element, the same in all lanes; `left`: elements from there to the tensor's end, as far as
// they are accessed through the descriptor.
template <int W>
__device__ __forceinline__ Rows rows_of(const void* chunk, int32_t left) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(chunk), 0, (left & ~3) * W, kBufferRaw);
}

// Row r, lane `tid` of it: elements 4 tid .. 4 tid + 3.
template <int W, bool KEEP = false>
__device__ __forceinline__ void load_words(Rows rows, int r, uint32_t tid, uint32_t (&out)[4]) {
  const int off = (int)(tid * (4 * W)) + r * (kRowLanes * 4 * W);
  if constexpr (W == 4) {
    const v4u v = __builtin_amdgcn_raw_buffer_load_b128(rows, off, 0, KEEP ? 0 : kNonTemporal);
    out[0] = v.x; out[1] = v.y; out[2] = v.z; out[3] = v.w;
  } else {
    const v2u v = __builtin_amdgcn_raw_buffer_load_b64(rows, off, 0, KEEP ? 0 : kNonTemporal);
    out[0] = v.x; out[1] = v.y;
  }
}

// The last left % 4 elements of a chunk of `left` elements.
struct Tail {
  bool any;     // this wavefront has them (uniform)
  bool mine;    // this lane has one: element `at` of the chunk
  uint32_t at;
  uint32_t owner;  // the lane of 256 that would have them as its four elements of row `row`
  uint32_t row;
};
__device__ __forceinline__ Tail tail_of(int32_t left, uint32_t tid) {
  const uint32_t whole = (uint32_t)left & ~3u, lane = tid & 63u, owner = whole % (kRowLanes * 4) / 4;
  const bool any = (left & 3) != 0 && (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid / 64u)) == owner / 64u;
  return Tail{any, any && lane < ((uint32_t)left & 3u), whole + lane, owner, whole / (kRowLanes * 4)};
}

// Rows again, of fp32 elements at plain addresses, for kernels that read so many arrays that their descriptors would not fit
// the scalar registers; `left`: elements from the row's first one to the end (a full row if FULL).
template <bool FULL, bool KEEP = false>
__device__ __forceinline__ void load_row4(const float* row, uint32_t tid, int32_t left, uint32_t (&out)[4]) {
  v4u v{0, 0, 0, 0};
  if (FULL || (int32_t)(tid * 4) + 4 <= left) {
    const auto p = (const TA_GLOBAL v4u*)(as_global<char>(row) + tid * 16u);
    v = KEEP ? *p : __builtin_nontemporal_load(p);
  }
  out[0] = v.x; out[1] = v.y; out[2] = v.z; out[3] = v.w;
}
template <bool FULL>
__device__ __forceinline__ void store_row4(float* row, uint32_t tid, int32_t left, const uint32_t (&w)[4]) {
  if (!FULL && (int32_t)(tid * 4) + 4 > left) return;
  v4u v;
  v.x = w[0]; v.y = w[1]; v.z = w[2]; v.w = w[3];
  __builtin_nontemporal_store(v, (TA_GLOBAL v4u*)(as_global<char>(row) + tid * 16u));
}

// A lane's word of the tail: fp32, or a 16-bit element in the low half.  0 in the lanes without one.
template <int W>
__device__ __forceinline__ uint32_t load_tail(const void* chunk, const Tail& t) {
  uint32_t v = 0;
  if (t.mine) {
    const auto p = as_global<char>(chunk) + t.at * (uint32_t)W;
    v = W == 4 ? *(const TA_GLOBAL uint32_t*)p : (uint32_t)*(const TA_GLOBAL uint16_t*)p;
  }
  return v;
}
template <int DT>
__device__ __forceinline__ void store_tail(void* chunk, const Tail& t, uint32_t bits) {
  if (!t.mine) return;
  const auto p = as_global<char>(chunk) + t.at * (uint32_t)kWords<DT>;
  if constexpr (DT == kFP32) *(TA_GLOBAL uint32_t*)p = bits;
  else *(TA_GLOBAL uint16_t*)p = (uint16_t)(DT == kBF16 ? f32_to_bf16_bits(u2f(bits)) : f32_to_f16_bits(u2f(bits)));
}
template <int DT>
__device__ __forceinline__ uint32_t widen1(uint32_t w) {
  return DT == kFP32 ? w : DT == kBF16 ? w << 16 : f2u(f16_bits_to_f32(w));
}

// In place: words as loaded -> the four values' fp32 bit patterns.
template <int DT>
__device__ __forceinline__ void widen4(uint32_t (&w)[4]) {
  if constexpr (DT == kBF16) {
    w[3] = w[1] & 0xffff0000u; w[2] = w[1] << 16;
    w[1] = w[0] & 0xffff0000u; w[0] = w[0] << 16;
  } else if constexpr (DT == kFP16) {
    w[3] = f2u(f16_bits_to_f32(w[1] >> 16)); w[2] = f2u(f16_bits_to_f32(w[1] & 0xffffu));
    w[1] = f2u(f16_bits_to_f32(w[0] >> 16)); w[0] = f2u(f16_bits_to_f32(w[0] & 0xffffu));
  }
}

template <int DT>
__device__ __forceinline__ float load1(const void* base, int64_t idx) {
  if constexpr (DT == kFP32) return as_global<float>(base)[idx];
  const uint32_t h = as_global<uint16_t>(base)[idx];
  if constexpr (DT == kBF16) return bf16_bits_to_f32(h);
  return f16_bits_to_f32(h);
}

// In place: fp32 bit patterns -> words in the storage precision.
template <int DT>
__device__ __forceinline__ void narrow4(uint32_t (&w)[4]) {
  if constexpr (DT != kFP32) {
    uint32_t h[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) h[i] = (DT == kBF16) ? f32_to_bf16_bits(u2f(w[i])) : f32_to_f16_bits(u2f(w[i]));
    w[0] = h[0] | (h[1] << 16);
    w[1] = h[2] | (h[3] << 16);
  }
}

template <int W>
__device__ __forceinline__ void store_words(Rows rows, int r, uint32_t tid, const uint32_t (&w)[4]) {
  const int off = (int)(tid * (4 * W)) + r * (kRowLanes * 4 * W);
  if constexpr (W == 4) {
    v4u o;
    o.x = w[0]; o.y = w[1]; o.z = w[2]; o.w = w[3];
    __builtin_amdgcn_raw_buffer_store_b128(o, rows, off, 0, kNonTemporal);
  } else {
    v2u o;
    o.x = w[0]; o.y = w[1];
    __builtin_amdgcn_raw_buffer_store_b64(o, rows, off, 0, kNonTemporal);
  }
}

}  // namespace triaccel
