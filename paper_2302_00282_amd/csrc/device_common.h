// Device-side vocabulary shared by the gfx950 kernel sources: vector types, the element-type traits (fp32 / bf16
// storage, fp32 arithmetic), bf16 conversion, and the tile constants of the MFMA GEMM loops.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <atomic>
#include <type_traits>
#include "index_div.h"
#include "kernels.h"

namespace xenos {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;

struct bf16_t { uint16_t v; };

__device__ __forceinline__ float bf2f(uint16_t v) { return __uint_as_float(((uint32_t)v) << 16); }
// fp32 -> bf16, round-to-nearest-even: gfx950 converts in hardware (one packed instruction per two values)
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef __attribute__((ext_vector_type(2))) float f32x2_t;
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ __forceinline__ uint32_t f2bf2(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){lo, hi}, bf16x2_t));
}

template <typename T> struct Tr;
template <> struct Tr<float> {
  static constexpr int CE = 4;     // elements per 16-byte chunk
  static constexpr int BKE = kRowBytes / 4;   // reduction elements per step
  __device__ static __forceinline__ float ld(const void* p, long long i) { return ((const float*)p)[i]; }
  __device__ static __forceinline__ void st(void* p, long long i, float v) { ((float*)p)[i] = v; }
  __device__ static __forceinline__ void unpack(const u32x4_t& v, float* f) {
#pragma unroll
    for (int e = 0; e < 4; ++e) f[e] = __uint_as_float(v[e]);
  }
  __device__ static __forceinline__ u32x4_t pack(const float* f) {
    u32x4_t v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = __float_as_uint(f[e]);
    return v;
  }
};
template <> struct Tr<bf16_t> {
  static constexpr int CE = 8;
  static constexpr int BKE = kRowBytes / 2;
  __device__ static __forceinline__ float ld(const void* p, long long i) { return bf2f(((const uint16_t*)p)[i]); }
  __device__ static __forceinline__ void st(void* p, long long i, float v) { ((uint16_t*)p)[i] = f2bf(v); }
  __device__ static __forceinline__ void unpack(const u32x4_t& v, float* f) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      f[2 * e] = __uint_as_float(v[e] << 16);
      f[2 * e + 1] = __uint_as_float(v[e] & 0xffff0000u);
    }
  }
  __device__ static __forceinline__ u32x4_t pack(const float* f) {
    u32x4_t v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = f2bf2(f[2 * e], f[2 * e + 1]);
    return v;
  }
};

// 16-byte loads through a buffer descriptor: a 32-bit byte offset from a wavefront-uniform base; an offset beyond the window's `bytes`
// (kNoLoad, or any with bytes = 0) reads zeros and no memory.  A masked element costs neither a branch nor a selection, and a loop can
// issue the same loads on every turn: behind a branch around them the compiler has to assume the path with the fewest loads in flight
// and waits for all of them.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
constexpr unsigned kNoLoad = 0xffffffffu, kWindow = 0xffffff00u;     // (kWindow: the largest, for offsets that the host has bounded)
__device__ __forceinline__ rsrc_t make_window(const void* base, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00027000);
}
// (soff is not part of what is compared with the window: 0, or inside it together with off)
__device__ __forceinline__ u32x4_t load_window(rsrc_t w, unsigned off, unsigned soff = 0) {
  return __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(w, (int)off, __builtin_amdgcn_readfirstlane((int)soff), 0));
}
// off or nothing.  (Without the barrier the compiler makes a branch of the selection, with a load on either side.)
__device__ __forceinline__ u32x4_t load_window_if(rsrc_t w, bool ok, unsigned off) {
  unsigned o = ok ? off : kNoLoad;
  asm volatile("" : "+v"(o));
  return load_window(w, o);
}

// max(a, b).  `fmaxf` must quiet signalling NaNs, which costs an extra `v_max x, x, x` per operand whose origin the compiler
// cannot see: values moved between lanes by DPP or unpacked from bf16 with bit operations, i.e. every operand of the
// pooling reductions (two thirds of their instructions).  fmx_raw is the bare instruction for those places; NaN inputs are
// outside the contract of the library.
__device__ __forceinline__ float fmx(float a, float b) { return __builtin_fmaxf(a, b); }
__device__ __forceinline__ float fmx_raw(float a, float b) {
  float r;
  asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// ReLU as a maximum, or nothing: max(y, NaN) is y for every y, infinite ones too (the lowest finite number as a floor would
// replace -infinity).  For fmx_raw: of fmaxf the compiler makes a maximum and a selection per value.
__device__ __forceinline__ float relu_floor(int relu) { return relu ? 0.f : __builtin_nanf(""); }
// the same maximum with the floor in a scalar register
__device__ __forceinline__ float fmx_floor(float y, float lo) {
  float r;
  asm("v_max_f32 %0, %1, %2" : "=v"(r) : "s"(lo), "v"(y));
  return r;
}

// Two-group channel shuffle done by a store: CE finished channels of a pixel (`mine`) and the same channels of the other
// part of the concat (`oth`) alternate in the output, `first` = mine at the even positions.  Two 16-byte stores.
template <typename T>
__device__ __forceinline__ void ileave_store(T* dst, const u32x4_t& mine, const u32x4_t& oth, bool first) {
  u32x4_t w[2];
  if (sizeof(T) == 2) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const uint32_t m = (mine[e >> 1] >> ((e & 1) * 16)) & 0xffffu, o = (oth[e >> 1] >> ((e & 1) * 16)) & 0xffffu;
      w[e >> 2][e & 3] = first ? (m | (o << 16)) : (o | (m << 16));
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      w[e >> 1][(e & 1) * 2] = first ? mine[e] : oth[e];
      w[e >> 1][(e & 1) * 2 + 1] = first ? oth[e] : mine[e];
    }
  }
  *(u32x4_t*)dst = w[0];
  *(u32x4_t*)(dst + Tr<T>::CE) = w[1];
}

// The argument structs are some 600 bytes, ten lines of the constant cache, and the compiler fetches their members in the
// order of use: four or more dependent round trips before the first tensor is touched.  Called first in a kernel, this
// requests a word of every line at once and waits for them together, so that later reads hit (MobileNet batch 1, bf16, 17
// launches: 118.5 -> 108.1 us; ShuffleNet batch 32, 39 launches: 526 -> 509 us).
template <int BYTES>
__device__ __forceinline__ void fetch_args(const void* ka) {
  static_assert(BYTES > 0x40 && BYTES <= 640 && !(BYTES > 192 && BYTES <= 0x240), "a request per line, none past the struct");
  uint32_t w;
  if constexpr (BYTES > 128 && BYTES <= 192)
    asm volatile("s_load_dword %0, %1, 0x0\n s_load_dword %0, %1, 0x40\n s_load_dword %0, %1, 0x80\n s_waitcnt lgkmcnt(0)" : "=&s"(w) : "s"(ka));
  else if constexpr (BYTES > 512)
    asm volatile("s_load_dword %0, %1, 0x0\n s_load_dword %0, %1, 0x40\n s_load_dword %0, %1, 0x80\n s_load_dword %0, %1, 0xc0\n"
                 "s_load_dword %0, %1, 0x100\n s_load_dword %0, %1, 0x140\n s_load_dword %0, %1, 0x180\n s_load_dword %0, %1, 0x1c0\n"
                 "s_load_dword %0, %1, 0x200\n s_load_dword %0, %1, 0x240\n s_waitcnt lgkmcnt(0)" : "=&s"(w) : "s"(ka));
  else
    asm volatile("s_load_dword %0, %1, 0x0\n s_load_dword %0, %1, 0x40\n s_waitcnt lgkmcnt(0)" : "=&s"(w) : "s"(ka));
}
#define FETCH_ARGS(T) fetch_args<(int)sizeof(T)>((const void*)__builtin_amdgcn_kernarg_segment_ptr())

// division by a run-time integer that many indices share (index_div.h)
struct SmallDiv {
  int d;
  float r;
  __device__ __forceinline__ explicit SmallDiv(int d_) : d(d_), r(__builtin_amdgcn_rcpf((float)d_)) {}
  __device__ __forceinline__ int operator()(int n) const { return small_quotient(n, r); }
};
struct AnyDiv {
  int d;
  float r;
  __device__ __forceinline__ explicit AnyDiv(int d_) : d(d_), r(__builtin_amdgcn_rcpf((float)d_)) {}
  __device__ __forceinline__ int operator()(int n) const { return any_quotient(n, d, r); }
};
// n / d of wavefront-uniform values of any size
__device__ __forceinline__ int uniform_div(int n, int d) {
  return __builtin_amdgcn_readfirstlane(n < kSmallDiv ? SmallDiv(d)(n) : n / d);
}

// n / d of wavefront-uniform values by the host's multiplier, one scalar multiplication (the reciprocal on the vector unit, its conversions and
// the way back were some 90 cycles each, three of them in a row before a tile's first request); mul = 0: by the reciprocal all the same
__device__ __forceinline__ int tile_div(int n, int d, unsigned mul) {
  if (mul) return (int)host_quotient((unsigned)n, mul);
  asm volatile("" : "+s"(d));                          // (nothing of the division is worked out ahead, for calls that need none)
  return uniform_div(n, d);
}

// Dynamic LDS of a kernel whose launches differ in their need: its limit is raised once, to all of a unit's memory.  (Raised to what
// the launch at hand needs, two threads' first launches could leave the smaller limit behind.)
constexpr int kLdsPerUnit = 160 * 1024;
template <typename F>
inline hipError_t raise_lds_limit(F* kernel, std::atomic<bool>& raised) {
  if (raised.load(std::memory_order_acquire)) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsPerUnit);
  if (e == hipSuccess) raised.store(true, std::memory_order_release);
  return e;
}

constexpr int NT = 256;          // threads per workgroup (4 wavefronts of 64)
constexpr int ROWB = kRowBytes;  // data bytes per tile row per reduction step
constexpr int CPR = ROWB / 16;   // 16-byte chunks per tile row
constexpr int KG = ROWB / 32;    // k-groups (one MFMA fragment pair each) per step
constexpr int LDS_ROW = ROWB + 16;   // row pitch in LDS: an odd number of 16-byte slots, so consecutive rows hit distinct slots
constexpr int NUM_XCD = 8;

__host__ __device__ constexpr int cmax(int a, int b) { return a > b ? a : b; }

}  // namespace xenos
