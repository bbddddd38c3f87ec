// The reduction of a tile shared out over the wavefronts of a workgroup (device code of the wave kernels): the chains of few pixels in bf16, and
// every dense chain in fp32, whose products are made on the bf16 MFMAs here.
//
// At batch 1 a chain is 30 to 250 workgroups whose time is a chain of latencies, not bytes or MFMAs.  With all four wavefronts on one
// tile step by step (request into registers, write to LDS, barrier, read fragments, multiply) a step of 128 bytes per row takes 690
// cycles, of which the MFMAs are 128 and the 16 KB from the cache 256.  Here a wavefront owns every fourth step of the tile's
// reduction: it brings the operands of several steps straight into LDS of its own (buffer loads that write LDS: no registers, no LDS
// writes to issue), waits for the oldest only and multiplies, with no barrier until the four partial tiles are added at the end.
#pragma once
#include "device_common.h"

namespace xenos {

// LDS rows of 128 bytes, 16-byte slot s of row r holds chunk s ^ wave_swizzle(r): the sixteen lanes that one pass of a fragment read
// serves (rows that differ mod 16) then hit sixteen different slots of the 256 bytes that LDS reads at a time.  (A load that writes LDS
// puts its 64 lanes' 16 bytes behind one another, so rows cannot be padded; what a lane may choose is the chunk it loads.)
__device__ __forceinline__ int wave_swizzle(int row) { return (row >> 1) & 7; }

// wait until at most N of this wavefront's memory requests are on their way (they complete in order)
template <int N>
__device__ __forceinline__ void wait_requests() {
  static_assert(N >= 0 && N < 64, "the counter has six bits");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0f70);
  asm volatile("" ::: "memory");
}

typedef __attribute__((address_space(3))) void* lds_ptr_t;
__device__ __forceinline__ void load_to_lds(rsrc_t w, unsigned char* dst, unsigned off, unsigned soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(w, (lds_ptr_t)dst, 16, (int)off, (int)soff, 0, 0);
}

// A wavefront's share of a tile of 32 * NB rows x 32 * NB channels (transposed: accumulator rows are channels, columns the tile's rows).  This is bf16; fp32 below
template <typename T, int NB>
struct WaveTile {
  static_assert(sizeof(T) == 2, "fp32 has a form of its own");
  static constexpr int EDGE = 32 * NB;
  static constexpr int STAGE = 2 * EDGE * ROWB;        // LDS of a step: pixel rows, then channel rows
  static constexpr int LOADS = 2 * EDGE / 8;           // requests of a step
  static constexpr int MAX_STAGES = NB == 1 ? 4 : 2;
  static constexpr int SLOTS = EDGE / 4;               // four channels each, of a row of the partial tile in LDS
  static_assert(EDGE * EDGE * 4 <= STAGE && LOADS * (MAX_STAGES - 1) < 64, "the partial tile takes the place of a stage; waits can count the requests");

  // n steps, `stages` (1 .. MAX_STAGES) of them on their way at a time; request(i, dst) issues LOADS requests for step i of this wavefront
  template <typename Request>
  __device__ __forceinline__ static void begin(int n, int stages, unsigned char* s_w, Request request) {
#pragma unroll 1
    for (int d = 0; d < stages && d < n; ++d) request(d, s_w + d * STAGE);
  }
  template <typename Request>
  __device__ __forceinline__ static void finish(int n, int stages, unsigned char* s_w, Request request) {
    const int lane = threadIdx.x & 63, l31 = lane & 31, lhalf = lane >> 5;
    // (row l31 of every block of 32 has the same swizzle; k-group kg is chunks 2 kg and 2 kg + 1, the lane's half chooses)
    int slot[KG];
#pragma unroll
    for (int kg = 0; kg < KG; ++kg) slot[kg] = l31 * ROWB + (((2 * kg + lhalf) ^ wave_swizzle(l31)) * 16);
    f32x16_t acc[NB][NB];                                              // [pixel block][channel block]
#pragma unroll
    for (int r = 0; r < NB; ++r)
#pragma unroll
      for (int c = 0; c < NB; ++c)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[r][c][e] = 0.f;
    unsigned char* s = s_w;
    int st = 0;
    // (the fragments of a step are read behind the multiplications of the step before it: requested ahead of them, in twice the registers, they
    // cost 4 to 7 % of the chains' time)
#pragma unroll 1
    for (int i = 0; i < n; ++i) {
      const int behind = n - 1 - i < stages - 1 ? n - 1 - i : stages - 1;   // (uniform) steps requested behind this one
      if (MAX_STAGES > 3 && behind >= 3) wait_requests<(MAX_STAGES > 3 ? 3 : 0) * LOADS>();
      else if (MAX_STAGES > 2 && behind == 2) wait_requests<(MAX_STAGES > 2 ? 2 : 0) * LOADS>();
      else if (behind == 1) wait_requests<LOADS>();
      else wait_requests<0>();
      u32x4_t fa[NB][KG], fb[NB][KG];
#pragma unroll
      for (int kg = 0; kg < KG; ++kg)
#pragma unroll
        for (int r = 0; r < NB; ++r) {
          fa[r][kg] = *(const u32x4_t*)(s + r * 32 * ROWB + slot[kg]);
          fb[r][kg] = *(const u32x4_t*)(s + (NB + r) * 32 * ROWB + slot[kg]);
        }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");               // the stage has been read: it may be written again
      if (i + stages < n) request(i + stages, s);
#pragma unroll
      for (int kg = 0; kg < KG; ++kg)
#pragma unroll
        for (int r = 0; r < NB; ++r)
#pragma unroll
          for (int c = 0; c < NB; ++c)
            acc[r][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, fb[c][kg]), __builtin_bit_cast(bf16x8_t, fa[r][kg]), acc[r][c], 0, 0, 0);
      if (++st == stages) { st = 0; s = s_w; } else { s += STAGE; }
    }
    // the partial tile, [row][channel], in this wavefront's own LDS; four channels of row r lie in slot (their number ^ r)
#pragma unroll
    for (int r = 0; r < NB; ++r)
#pragma unroll
      for (int c = 0; c < NB; ++c)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *(f32x4_t*)(s_w + (r * 32 + l31) * EDGE * 4 + (((c * 8 + g * 2 + lhalf) ^ l31) & (SLOTS - 1)) * 16) =
              f32x4_t{acc[r][c][4 * g], acc[r][c][4 * g + 1], acc[r][c][4 * g + 2], acc[r][c][4 * g + 3]};
  }
  // channels 4 c4 .. 4 c4 + 3 of a row, the wavefronts' partial tiles (wave_bytes apart) added in their order
  __device__ __forceinline__ static f32x4_t sum(const unsigned char* s, int wave_bytes, int row, int c4) {
    f32x4_t v[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) v[w] = *(const f32x4_t*)(s + w * wave_bytes + row * EDGE * 4 + ((c4 ^ row) & (SLOTS - 1)) * 16);
    return ((v[0] + v[1]) + v[2]) + v[3];
  }
};

// Three bf16 values whose sum is x * kWavePartScale (each rounds what the ones before it leave; the third is exact, eight of the 24 bits), whatever x is
// below 2^103.  Infinite values, and finite ones that become so, leave NaN.
struct Split8 { bf16x8_t hi, mid, lo; };
__device__ __forceinline__ Split8 split8(const u32x4_t& a, const u32x4_t& b) {
  u32x4_t p[3];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float x0 = __uint_as_float(i < 2 ? a[2 * i] : b[2 * i - 4]) * kWavePartScale, x1 = __uint_as_float(i < 2 ? a[2 * i + 1] : b[2 * i - 3]) * kWavePartScale;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const uint32_t u = f2bf2(x0, x1);
      p[q][i] = u;
      x0 -= __uint_as_float(u << 16);
      x1 -= __uint_as_float(u & 0xffff0000u);
    }
  }
  return Split8{__builtin_bit_cast(bf16x8_t, p[0]), __builtin_bit_cast(bf16x8_t, p[1]), __builtin_bit_cast(bf16x8_t, p[2])};
}

// fp32 tiles on the bf16 MFMAs, which multiply at sixteen times the rate of the fp32 ones: both operands are split into three bf16 values whose sum they
// are, the weights when they are packed, the pixels as fragments are read, and six of the nine products are summed in fp32 (the three left out are below
// 2^-24 of the product).  The five small ones have sums of their own, so that the large ones are rounded once in sixteen products: against 64 bits dot products
// of 16 to 4608 random numbers are off by 3.2e-8 to 4.2e-7 of their norm, half or less of the fp32 MFMAs' 5.5e-8 to 1.2e-6.  A step is twelve MFMAs of 32
// cycles instead of sixteen of 64.  The image of a step of the weights lies in memory as in LDS: [hi, mid, lo][32 channels][64 bytes], 16-byte slot s of
// row r holds chunk s ^ (r / 4 % 4).  Sums that are not finite are for the caller to work out again: those of an infinite operand or one that is not a number, and,
// products being 2^48 times too large, any beyond 2^79 and of a pixel or weight from 2^103 on.  (The scale costs a multiplication a pixel value: SqueezeNet batch 32
// 426 -> 432 us, MobileNet batch 1 95.5 -> 96.7; without it operands below 2^-110 had fewer than 24 bits, 1e-38 ten.)
template <int NB>
struct WaveTile<float, NB> {
  static constexpr int EDGE = 32 * NB, ROWS_A = EDGE * ROWB, PLANE = 32 * 64, BLOCK = 3 * PLANE;
  static constexpr int STAGE = NB * (int)kWaveStageF32; // pixel rows, then the three planes of the rows of each 32 channels
  static constexpr int LOADS = (ROWS_A + NB * BLOCK) / 1024;
  static constexpr int MAX_STAGES = NB == 1 ? 3 : 2, SLOTS = EDGE / 4;
  static_assert(STAGE == ROWS_A + NB * BLOCK && EDGE * EDGE * 4 <= STAGE && LOADS * (MAX_STAGES - 1) < 64, "the partial tile takes the place of a stage; waits can count the requests");

  template <typename Request>
  __device__ __forceinline__ static void begin(int n, int stages, unsigned char* s_w, Request request) {
#pragma unroll 1
    for (int d = 0; d < stages && d < n; ++d) request(d, s_w + d * STAGE);
  }
  template <typename Request>
  __device__ __forceinline__ static void finish(int n, int stages, unsigned char* s_w, Request request) {
    const int lane = threadIdx.x & 63, l31 = lane & 31, lhalf = lane >> 5;
    // the lane's eight values of a pixel in either half of a step, 16 bytes at a time, and of weights: chunks 4 g + 2 lhalf + 0 and 1, and 2 g + lhalf
    // (their slots differ in one bit of the address, stages being multiples of 1 KB; worked out by step, for want of registers)
    const uint32_t aslot = (uint32_t)(uintptr_t)(lds_ptr_t)s_w + l31 * ROWB + ((2 * lhalf) ^ wave_swizzle(l31)) * 16;
    const uint32_t wslot = (uint32_t)(uintptr_t)(lds_ptr_t)s_w + ROWS_A + l31 * 64 + (lhalf ^ ((l31 >> 2) & 3)) * 16;
    typedef const __attribute__((address_space(3))) u32x4_t* lds_vec_t;
    f32x16_t acc[NB][NB], small[NB][NB];                               // [pixel block][channel block]
#pragma unroll
    for (int r = 0; r < NB; ++r)
#pragma unroll
      for (int c = 0; c < NB; ++c)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[r][c][e] = small[r][c][e] = 0.f;
    unsigned char* s = s_w;
    int st = 0;
#pragma unroll 1
    for (int i = 0; i < n; ++i) {
      const int behind = n - 1 - i < stages - 1 ? n - 1 - i : stages - 1;   // (uniform) steps requested behind this one
      if (MAX_STAGES > 2 && behind == 2) wait_requests<(MAX_STAGES > 2 ? 2 : 0) * LOADS>();
      else if (behind == 1) wait_requests<LOADS>();
      else wait_requests<0>();
      u32x4_t a[2][NB][2], w[2][NB][3];
      auto read = [&](int g) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < NB; ++r) {
#pragma unroll
          for (int q = 0; q < 2; ++q) a[g][r][q] = *(lds_vec_t)(uintptr_t)(((aslot + (uint32_t)(s - s_w)) ^ (uint32_t)(g * 64 + q * 16)) + r * 32 * ROWB);
#pragma unroll
          for (int q = 0; q < 3; ++q) w[g][r][q] = *(lds_vec_t)(uintptr_t)(((wslot + (uint32_t)(s - s_w)) ^ (uint32_t)(g * 32)) + r * BLOCK + q * PLANE);
        }
      };
      read(0);
      if constexpr (NB == 1) read(1);
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        if (g == 0 && NB == 1) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (g == 1) {
          if constexpr (NB > 1) {
            read(1);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          }
          // the stage has been read: it may be written again (asked for here, where fewer registers hold what was read)
          if (i + stages < n) request(i + stages, s);
        }
        Split8 x[NB];
#pragma unroll
        for (int r = 0; r < NB; ++r) x[r] = split8(a[g][r][0], a[g][r][1]);
#pragma unroll
        for (int r = 0; r < NB; ++r)
#pragma unroll
          for (int c = 0; c < NB; ++c) {
            const bf16x8_t hi = __builtin_bit_cast(bf16x8_t, w[g][c][0]), mid = __builtin_bit_cast(bf16x8_t, w[g][c][1]), lo = __builtin_bit_cast(bf16x8_t, w[g][c][2]);
            small[r][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lo, x[r].hi, small[r][c], 0, 0, 0);
            acc[r][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(hi, x[r].hi, acc[r][c], 0, 0, 0);
            small[r][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(mid, x[r].hi, small[r][c], 0, 0, 0);
            small[r][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(mid, x[r].mid, small[r][c], 0, 0, 0);
            small[r][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(hi, x[r].mid, small[r][c], 0, 0, 0);
            small[r][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(hi, x[r].lo, small[r][c], 0, 0, 0);
          }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (++st == stages) { st = 0; s = s_w; } else { s += STAGE; }
    }
#pragma unroll
    for (int r = 0; r < NB; ++r)
#pragma unroll
      for (int c = 0; c < NB; ++c)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x16_t &v = acc[r][c], &m = small[r][c];
          *(f32x4_t*)(s_w + (r * 32 + l31) * EDGE * 4 + (((c * 8 + g * 2 + lhalf) ^ l31) & (SLOTS - 1)) * 16) =
              f32x4_t{v[4 * g] + m[4 * g], v[4 * g + 1] + m[4 * g + 1], v[4 * g + 2] + m[4 * g + 2], v[4 * g + 3] + m[4 * g + 3]};
        }
  }
  __device__ __forceinline__ static f32x4_t sum(const unsigned char* s, int wave_bytes, int row, int c4) {
    f32x4_t v[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) v[w] = *(const f32x4_t*)(s + w * wave_bytes + row * EDGE * 4 + ((c4 ^ row) & (SLOTS - 1)) * 16);
    return (((v[0] + v[1]) + v[2]) + v[3]) * (1.f / (kWavePartScale * kWavePartScale));
  }
};
// element i of a step of row `row` of 32 channels, out of the packed image of that step
__device__ __forceinline__ float wave_weight_f32(const unsigned char* step, int row, int i) {
  const uint16_t* p = (const uint16_t*)(step + row * 64 + (((i >> 3) ^ ((row >> 2) & 3)) * 16)) + (i & 7);
  if (p[0] == kWaveWholeWeight) return __uint_as_float((uint32_t)p[1024] << 16 | p[2048]);
  return ((bf2f(p[0]) + bf2f(p[1024])) + bf2f(p[2048])) * (1.f / kWavePartScale);
}
__device__ __forceinline__ bool all_finite(const f32x4_t& v) {
  uint32_t e = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) e |= (__float_as_uint(v[i]) & 0x7f800000u) == 0x7f800000u ? 1u : 0u;
  return e == 0;
}

}  // namespace xenos
