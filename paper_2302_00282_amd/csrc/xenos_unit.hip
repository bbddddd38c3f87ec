// gfx950 (CDNA4) kernel of a depthwise-separable unit as one chain (Table 1, ConvX -> ConvY twice; Section 2.2):
//
//  unit_kernel   pointwise (1x1) chain -> depthwise 3x3 chain -> pointwise chain, both intermediate tensors on chip.
//
// A workgroup owns TH x TW output pixels of one image and ALL output channels: the depthwise convolution works per channel,
// but the second pointwise convolution sums over all of them.  It stages the input block (the pixels the tile's windows
// cover, all input channels) in LDS, runs the first GEMM of the positions inside the map into the LDS block the stencil reads
// (rounded to the storage type as a stored tensor would be; positions outside the map stay zero, the padding of the depthwise
// convolution; neighbouring tiles recompute the shared border), runs the stencil into the operand panel of the second GEMM,
// and that GEMM's epilogue stores the output, alternating with the other half of a shuffled concat where the unit ends in one.
//
// Bound: latency.  As two launches (1x1 convolution; depthwise -> pointwise, whose depthwise panel every 64-channel tile of the
// output recomputed) a 176-channel 14x14 unit at batch 32 took 8.4 + 18.2 us for 0.8 GFLOP and 7 MB; all output channels in
// one workgroup take the recomputation out, and both weight matrices, packed in fragment order, go from the cache straight
// into the registers of the wavefront that multiplies them, UN_RING k-groups ahead: no barrier inside a GEMM, four per tile.
// A network of such units (ShuffleNet graph, batch 32, bf16): 509 -> 319 us.  Timestamps of the first version (176 channels,
// cycles): input block 5.0 k, first GEMM 5.2 k, stencil 2.8 k, second GEMM and stores 6.5 k.  So the weights travel a phase ahead: the
// first GEMM's ring is requested behind the input block's first loads, the second one's as the first one's is used up (it arrives
// behind the stencil), and the other half of a shuffled concat ahead of the reduction it waits for: 314.3 -> 308.0 us.  The rest of that
// latency is all workgroups reading the same 60 to 250 KB of weights.  Kept for 12 k-groups only, and what depends on the thread's index
// computed per tile: requesting all weights and the depthwise weights at the start was slower (spilled: 371 against 352 us).
#include "device_common.h"

namespace xenos {

constexpr int UN_NT = 512, UN_NW = UN_NT / 64;   // eight wavefronts
constexpr int UN_RING = 12;                      // weight fragments in flight per wavefront: 12 KB

// LDS row of c channels: whole 32-byte k-groups and one odd 16-byte slot
__host__ __device__ constexpr int unit_pitch(int c, int esz) { return (c * esz + 31) / 32 * 32 + 16; }
__host__ __device__ constexpr int unit_stg_pitch(int esz) { return 32 * esz + 16; }
// input block, later the stencil's panel | block the stencil reads, later the staging slices of the wavefronts
__host__ __device__ constexpr int unit_lds_a(int positions, int pixels, int c1, int c, int esz) {
  return cmax(positions * unit_pitch(c1, esz), pixels * unit_pitch(c, esz));
}
__host__ __device__ constexpr int unit_lds_b(int positions, int c, int esz) {
  return cmax(positions * unit_pitch(c, esz), UN_NW * 32 * unit_stg_pitch(esz));
}

// A pointer the compiler takes as new at this place: addresses computed from it stay inside the tile loop, as a wavefront-uniform
// base and a 32-bit lane offset.  (Hoisted out of the loop as 64-bit lane addresses they were spilled.)
typedef const __attribute__((address_space(1))) unsigned char* gptr_t;
__device__ __forceinline__ gptr_t here(const void* p) {
  uint64_t v = (uint64_t)p;
  asm volatile("" : "+s"(v));
  return (gptr_t)v;
}
// The thread's index, taken as new likewise
__device__ __forceinline__ int thread_here() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}
__device__ __forceinline__ u32x4_t ld16(gptr_t base, unsigned off) { return *(const __attribute__((address_space(1))) u32x4_t*)(base + off); }

// The weight fragments of a unit_gemm: w as [block of 32 channels][kgs][lane] of 16 bytes, nkg of the kgs k-groups in use.  Part u is 64
// rows x 32 channels and works with block u % ncb; a k-group past the end, and every one of a part past the end, reads no memory.
struct UnitWeights {
  const void* w;
  int kgs, nkg, ncb, parts;
  unsigned mul;                                        // multiplier of quotients by ncb (never 0: a block of all channels is in LDS)
  __device__ __forceinline__ UnitWeights(const void* w_, int kgs_, int nkg_, int ncb_, unsigned mul_, int nrows)
      : w(w_), kgs(kgs_), nkg(nkg_), ncb(ncb_), parts(ncb_ * ((nrows + 63) / 64)), mul(mul_) {}
  __device__ __forceinline__ rsrc_t window(int u) const {
    const int cb = u - (int)host_quotient((unsigned)u, mul) * ncb;
    return make_window((const unsigned char*)w + (long long)cb * kgs * 1024, u < parts ? nkg * 1024u : 0u);
  }
};
// k-groups 0 .. UN_RING - 1 of a part
__device__ __forceinline__ void unit_request(rsrc_t wp, u32x4_t (&rb)[UN_RING]) {
  const unsigned off = (thread_here() & 63) * 16u;
#pragma unroll
  for (int d = 0; d < UN_RING; ++d) rb[d] = load_window(wp, off + d * 1024u);
}

// Transposed GEMM of `nrows` LDS rows (pitch bytes apart) with the blocks of `w`, a wavefront per part.  rb holds the requested
// fragments of the wavefront's first part; as a part's last ones are used up, those of its next part are requested, behind the last
// part those of `next` (NEXT; otherwise none: empty requests pass through the data path behind real ones, up to 0.7 us a tile).  pre(block, row0) runs before a part's reduction, epi(block, row0, half, acc) receives each finished 32 x 32
// half of it: lane = row row0 + l31, channels 8 g + 4 lhalf + (0..3) of the block in acc[4 g ..].
template <typename T, bool NEXT, typename PreFn, typename EpiFn>
__device__ __forceinline__ void unit_gemm(const UnitWeights& w, u32x4_t (&rb)[UN_RING], rsrc_t next, const unsigned char* s_rows, int pitch, int nrows, PreFn pre, EpiFn epi) {
  const unsigned lane = thread_here() & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l31 = (int)lane & 31, lhalf = (int)lane >> 5;
  const int nkg = w.nkg, ncb = w.ncb;
  if (NEXT && wave >= w.parts) unit_request(next, rb);
#pragma unroll 1
  for (int u = wave; u < w.parts; u += UN_NW) {
    const int rg = (int)host_quotient((unsigned)u, w.mul), cb = u - rg * ncb, row0 = rg * 64;
    const bool two = row0 + 32 < nrows;                            // (uniform)
    const rsrc_t wp = w.window(u), wn = u + UN_NW < w.parts ? w.window(u + UN_NW) : next;
    pre(cb, row0);
    // (rows past the end read the last row; their results are not stored)
    const unsigned char* pa0 = s_rows + (row0 + l31 < nrows ? row0 + l31 : nrows - 1) * pitch + lhalf * 16;
    const unsigned char* pa1 = s_rows + (row0 + 32 + l31 < nrows ? row0 + 32 + l31 : nrows - 1) * pitch + lhalf * 16;
    f32x16_t acc0, acc1;
#pragma unroll
    for (int e = 0; e < 16; ++e) { acc0[e] = 0.f; acc1[e] = 0.f; }
    // N k-groups from k0 + d0 on: their fragments are read before the first MFMA
    auto block = [&](int k0, int d0, auto NC) __attribute__((always_inline)) {
      constexpr int N = decltype(NC)::value;
      u32x4_t fa0[N], fa1[N];
#pragma unroll
      for (int d = 0; d < N; ++d) {
        fa0[d] = *(const u32x4_t*)(pa0 + (k0 + d0 + d) * 32);
        fa1[d] = *(const u32x4_t*)(pa1 + (k0 + d0 + d) * 32);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int d = 0; d < N; ++d) {
        if constexpr (sizeof(T) == 2) {
          acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, rb[d0 + d]), __builtin_bit_cast(bf16x8_t, fa0[d]), acc0, 0, 0, 0);
          acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, rb[d0 + d]), __builtin_bit_cast(bf16x8_t, fa1[d]), acc1, 0, 0, 0);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) acc0 = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(rb[d0 + d][e]), __uint_as_float(fa0[d][e]), acc0, 0, 0, 0);
          if (two) {
#pragma unroll
            for (int e = 0; e < 4; ++e) acc1 = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(rb[d0 + d][e]), __uint_as_float(fa1[d][e]), acc1, 0, 0, 0);
          }
        }
      }
    };
    const bool more = NEXT || u + UN_NW < w.parts;                 // (uniform)
    auto round = [&](int k0, auto MORE) __attribute__((always_inline)) {
#pragma unroll
      for (int d0 = 0; d0 < UN_RING; d0 += 4) {
        if (decltype(MORE)::value || k0 + d0 + 4 <= nkg) {         // (uniform)
          block(k0, d0, std::integral_constant<int, 4>());
        } else {
#pragma unroll
          for (int d = 0; d < 3; ++d)
            if (k0 + d0 + d < nkg) block(k0, d0 + d, std::integral_constant<int, 1>());
        }
        if (decltype(MORE)::value || more) {
#pragma unroll
          for (int d = d0; d < d0 + 4; ++d)
            rb[d] = decltype(MORE)::value ? load_window(wp, lane * 16u + (unsigned)(k0 + UN_RING + d) * 1024u) : load_window(wn, lane * 16u + d * 1024u);
        }
      }
    };
    int k0 = 0;
#pragma unroll 1
    for (; k0 + UN_RING < nkg; k0 += UN_RING) round(k0, std::true_type());
    round(k0, std::false_type());
    epi(cb, row0, 0, acc0);
    if (two) epi(cb, row0 + 32, 1, acc1);
  }
}

template <typename T>
__global__ __launch_bounds__(UN_NT, 2) void unit_kernel(const ConvArgs a) {
  FETCH_ARGS(ConvArgs);
  using tr = Tr<T>;
  constexpr int CE = tr::CE, ESZ = (int)sizeof(T);
  constexpr int STP = unit_stg_pitch(ESZ), G = 32 * ESZ / 16, STG_IT = 32 * G / 64;
  extern __shared__ __align__(16) unsigned char smem[];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const u32x4_t z = {0u, 0u, 0u, 0u};

  const int s = a.dw_stride, C = a.C, C1 = a.unit_C;
  const int PH = (a.th - 1) * s + 3, PWd = (a.tw - 1) * s + 3, P = PH * PWd, npx = a.th * a.tw;
  const int PX = unit_pitch(C1, ESZ), PM = unit_pitch(C, ESZ);
  unsigned char* s_x = smem;                                       // input block [position inside the map][C1], later [pixel][C]
  unsigned char* s_mid = smem + unit_lds_a(P, npx, C1, C, ESZ);    // [block position][C]
  unsigned char* s_stg = s_mid + wave * 32 * STP;
  const int tiles_sp = a.tiles_y * a.tiles_x;
  const int cgs = C / CE;                                          // stencil: a thread keeps its channel group, pgs pixels side by side
  const SmallDiv by_cgs(cgs), by_tw(a.tw);
  const int pgs = by_cgs(UN_NT);
  u32x4_t rb[UN_RING];                                             // weight fragments in flight

  for (int t = blockIdx.x; t < a.ntiles; t += gridDim.x) {
    const int tid = thread_here(), lane = tid & 63, l31 = lane & 31, lhalf = lane >> 5;
    const int pg = by_cgs(tid), cg = tid - pg * cgs;
    const bool dw_on = pg < pgs;
    const int n = tile_div(t, tiles_sp, a.q_sp), rr = t - n * tiles_sp, ty = tile_div(rr, a.tiles_x, a.q_tx), tx = rr - ty * a.tiles_x;
    const int oy0 = ty * a.th, ox0 = tx * a.tw;
    const int iy0 = oy0 * s - 1, ix0 = ox0 * s - 1;                // map position of block position (0, 0)
    const int y_lo = iy0 > 0 ? iy0 : 0, y_hi = iy0 + PH < a.dw_H ? iy0 + PH : a.dw_H;
    const int x_lo = ix0 > 0 ? ix0 : 0, x_hi = ix0 + PWd < a.dw_W ? ix0 + PWd : a.dw_W;
    const int wv = x_hi - x_lo, npos = (y_hi - y_lo) * wv;          // the part of the block inside the map (never empty)
    const SmallDiv by_wv(wv);
    const UnitWeights w1(a.fire_w[0], a.unit_kred * ESZ / 32, (C1 * ESZ + 31) / 32, (C + 31) / 32, a.q_c, npos);
    const UnitWeights w2(a.w, a.Kred_pad * ESZ / 32, (C * ESZ + 31) / 32, (a.K + 31) / 32, a.q_k, npx);

    // ---- the input block, all channels; k-groups are filled up with zeros ---------------------------------
    {
      const int cpr = (PX - 16) / 16, total = npos * cpr;          // (a fraction of the LDS: far below kSmallDiv)
      const SmallDiv by_cpr(cpr);
      const gptr_t src = here((const T*)a.in + (long long)n * a.in_sN + (long long)y_lo * a.in_sH + (long long)x_lo * a.in_sW);
      const int sH = (int)a.in_sH * ESZ, sW = (int)a.in_sW * ESZ;  // (an image takes less than 2 GB)
      constexpr int U = 4;                                         // requests before the first LDS write
      u32x4_t v[U];
      auto request = [&](int i0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int i = i0 + u * UN_NT < total ? i0 + u * UN_NT : total - 1;
          const int r = by_cpr(i), c = i - r * cpr, py = by_wv(r), px = r - py * wv;
          const bool ok = c * CE < C1;
          v[u] = ld16(src, (unsigned)(py * sH + px * sW + (ok ? c * 16 : 0)));
          if (!ok) v[u] = z;
        }
        __builtin_amdgcn_sched_barrier(0);
      };
      auto store = [&](int i0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int i = i0 + u * UN_NT, r = by_cpr(i), c = i - r * cpr;
          if (i < total) *(u32x4_t*)(s_x + r * PX + c * 16) = v[u];
        }
      };
      request(tid);
      unit_request(w1.window(wave), rb);                           // on their way while the block is written
      __builtin_amdgcn_sched_barrier(0);
      store(tid);
      for (int i0 = tid + U * UN_NT; i0 < total; i0 += U * UN_NT) {
        request(i0);
        store(i0);
      }
    }
    if (npos < P)                                                  // the zero padding of the depthwise convolution
      for (int i = tid; i < P * (PM / 16); i += UN_NT) *(u32x4_t*)(s_mid + i * 16) = z;
    __syncthreads();

    f32x4_t sc[4], sh[4];                                          // scale and shift of the lane's channels
    // ---- first pointwise chain, into the stencil's block ----------------------------------------------------
    unit_gemm<T, true>(w1, rb, w2.window(wave), s_x, PX, npos,
      [&](int cb, int) __attribute__((always_inline)) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          sc[g] = *(const f32x4_t*)(a.fire_scale[0] + cb * 32 + g * 8 + lhalf * 4);
          sh[g] = *(const f32x4_t*)(a.fire_shift[0] + cb * 32 + g * 8 + lhalf * 4);
        }
      },
      [&](int cb, int row0, int, const f32x16_t& acc) __attribute__((always_inline)) {
        const int m = row0 + l31;
        if (m >= npos) return;
        const int py = by_wv(m), px = m - py * wv;
        unsigned char* dst = s_mid + ((y_lo + py - iy0) * PWd + (x_lo + px - ix0)) * PM;
        const float lo = relu_floor(a.fire_relu[0]);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int c = cb * 32 + g * 8 + lhalf * 4;
          if (c >= C) continue;
          float y[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) y[e] = fmx_raw(acc[4 * g + e] * sc[g][e] + sh[g][e], lo);
          if constexpr (sizeof(T) == 2) {
            uint2 o;
            o.x = f2bf2(y[0], y[1]);
            o.y = f2bf2(y[2], y[3]);
            *(uint2*)(dst + c * 2) = o;
          } else {
            *(f32x4_t*)(dst + c * 4) = f32x4_t{y[0], y[1], y[2], y[3]};
          }
        }
      });
    const gptr_t dwp = here(a.dw_w);
    u32x4_t dww[9];                                                // this thread's depthwise weights, on their way over the barrier
#pragma unroll
    for (int t9 = 0; t9 < 9; ++t9) dww[t9] = ld16(dwp + t9 * C * ESZ, (unsigned)cg * 16u);
    __syncthreads();                                               // the block is complete, the input block is free

    // ---- depthwise chain, into the operand panel of the second GEMM -----------------------------------------
    if (dw_on) {
      float dsc[CE], dsh[CE];
#pragma unroll
      for (int e = 0; e < CE; e += 4) {
        *(f32x4_t*)&dsc[e] = *(const f32x4_t*)(a.dw_scale + cg * CE + e);
        *(f32x4_t*)&dsh[e] = *(const f32x4_t*)(a.dw_shift + cg * CE + e);
      }
      for (int q = pg; q < npx; q += pgs) {
        const int qy = by_tw(q), qx = q - qy * a.tw;
        const unsigned char* src = s_mid + ((qy * s) * PWd + qx * s) * PM + cg * 16;
        u32x4_t xr[9];
#pragma unroll
        for (int t9 = 0; t9 < 9; ++t9) xr[t9] = *(const u32x4_t*)(src + ((t9 / 3) * PWd + t9 % 3) * PM);
        float d[CE];
#pragma unroll
        for (int e = 0; e < CE; ++e) d[e] = 0.f;
#pragma unroll
        for (int t9 = 0; t9 < 9; ++t9) {
          float x[CE], w[CE];
          tr::unpack(xr[t9], x);
          tr::unpack(dww[t9], w);
#pragma unroll
          for (int e = 0; e < CE; ++e) d[e] = fmaf(x[e], w[e], d[e]);
        }
#pragma unroll
        for (int e = 0; e < CE; ++e) {
          const float y = d[e] * dsc[e] + dsh[e];
          d[e] = a.dw_relu ? fmx(y, 0.f) : y;
        }
        *(u32x4_t*)(s_x + q * PM + cg * 16) = tr::pack(d);
      }
    }
    if (C * ESZ % 32 != 0)                                         // the other half of the last k-group
      for (int q = tid; q < npx; q += UN_NT) *(u32x4_t*)(s_x + q * PM + C * ESZ) = z;
    __syncthreads();                                               // the panel is complete, the block is free

    // ---- second pointwise chain -------------------------------------------------------------------------------
    u32x4_t oth[2][STG_IT];                                        // the other half of the concat, requested ahead of the reduction
    // the output pixel of which the lane stores 16 bytes in round u of a half; false: none
    auto pixel = [&](int ln, int cb, int row, int u, long long& p) __attribute__((always_inline)) {
      const int idx = ln + u * 64, r = idx / G, g16 = idx - r * G;
      const int q = row + r, qy = by_tw(q), qx = q - qy * a.tw, oy = oy0 + qy, ox = ox0 + qx;
      p = (long long)oy * a.OW + ox;
      return q < npx && oy < a.OH && ox < a.OW && cb * 32 + g16 * CE < a.K;
    };
    auto other = [&](int cb, int row, int h) __attribute__((always_inline)) {
      if (!a.ileave) {                                             // (uniform: no shuffle, no addresses to work out)
#pragma unroll
        for (int u = 0; u < STG_IT; ++u) asm("" : "=v"(oth[h][u]));
        return;
      }
      const int ln = thread_here() & 63;
#pragma unroll
      for (int u = 0; u < STG_IT; ++u) {
        const int k0 = cb * 32 + (ln + u * 64) % G * CE;
        long long p;
        const bool ok = pixel(ln, cb, row, u, p);
        oth[h][u] = ok ? *(const u32x4_t*)((const T*)a.res + (long long)n * a.res_sN + p * a.res_sP + k0) : z;
      }
    };
    unit_gemm<T, false>(w2, rb, make_window(a.w, 0), s_x, PM, npx,
      [&](int cb, int row0) __attribute__((always_inline)) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          sc[g] = *(const f32x4_t*)(a.scale + cb * 32 + g * 8 + lhalf * 4);
          sh[g] = *(const f32x4_t*)(a.shift + cb * 32 + g * 8 + lhalf * 4);
        }
        if constexpr (sizeof(T) == 2) other(cb, row0, 0), other(cb, row0 + 32, 1);
      },
      [&](int cb, int row0, int h, const f32x16_t& acc) __attribute__((always_inline)) {
        // finished values change hands inside the wavefront only (LDS serves its requests in order)
        const float lo = relu_floor(a.relu);
        const int ln = thread_here() & 63, l31 = ln & 31, lhalf = ln >> 5;
        if constexpr (sizeof(T) != 2) other(cb, row0, h);          // (32 registers of both halves would be spilled)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int c = g * 8 + lhalf * 4;
          float y[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) y[e] = fmx_raw(acc[4 * g + e] * sc[g][e] + sh[g][e], lo);
          if constexpr (sizeof(T) == 2) {
            uint2 o;
            o.x = f2bf2(y[0], y[1]);
            o.y = f2bf2(y[2], y[3]);
            *(uint2*)(s_stg + l31 * STP + c * 2) = o;
          } else {
            *(f32x4_t*)(s_stg + l31 * STP + c * 4) = f32x4_t{y[0], y[1], y[2], y[3]};
          }
        }
#pragma unroll
        for (int u = 0; u < STG_IT; ++u) {
          const int idx = ln + u * 64, r = idx / G, g16 = idx - r * G;
          const u32x4_t mine = *(const u32x4_t*)(s_stg + r * STP + g16 * 16);
          const int k0 = cb * 32 + g16 * CE;
          long long p;
          if (!pixel(ln, cb, row0, u, p)) continue;
          T* dst = (T*)a.out + (long long)n * a.out_sN + p * a.out_sP + (a.ileave ? 2 * k0 : k0);
          if (a.ileave) ileave_store<T>(dst, mine, oth[h][u], a.ileave == 1);
          else *(u32x4_t*)dst = mine;
        }
      });
    __syncthreads();                                               // both regions are rewritten by the next tile
  }
}

size_t unit_lds_bytes(int th, int tw, int stride, int c1, int c, int esz) {
  const int positions = ((th - 1) * stride + 3) * ((tw - 1) * stride + 3);
  return (size_t)unit_lds_a(positions, th * tw, c1, c, esz) + unit_lds_b(positions, c, esz);
}

template <typename T>
static int launch_unit_t(const ConvArgs& a, hipStream_t st) {
  constexpr int ESZ = (int)sizeof(T), CE = Tr<T>::CE, BKE = Tr<T>::BKE;
  const int s = a.dw_stride;
  // what the kernel assumes, checked again on the host: a wrong shape would index outside the LDS block or the tensors (the caller's
  // output may lie at any element: the hardware takes 16-byte stores there)
  if (a.mode != M_FLAT || a.has_res || a.pool != POOL_NONE || a.ksplit >= 1 || a.kchunk || a.pair || a.fire || a.pwdw || !a.wfrag || !a.vec_out ||
      a.R != 1 || a.S != 1 || a.stride != 1 || a.pad != 0 || a.C % CE != 0 || a.K % CE != 0 || a.C < CE || a.K < CE || a.C / CE > UN_NT ||
      a.unit_C % CE != 0 || a.unit_C < CE || a.Kred_pad < (a.C + BKE - 1) / BKE * BKE || a.Kred_pad % BKE != 0 ||
      a.unit_kred < (a.unit_C + BKE - 1) / BKE * BKE || a.unit_kred % BKE != 0 || a.dw_k != 3 || a.dw_pad != 1 || (s != 1 && s != 2) ||
      !a.dw_w || !a.dw_scale || !a.dw_shift || !a.fire_w[0] || !a.fire_scale[0] || !a.fire_shift[0] ||
      a.OH != (a.dw_H + 2 - 3) / s + 1 || a.OW != (a.dw_W + 2 - 3) / s + 1 || a.th < 1 || a.tw < 1 ||
      a.tiles_y != (a.OH + a.th - 1) / a.th || a.tiles_x != (a.OW + a.tw - 1) / a.tw || a.tiles_n != 1 ||
      a.tiles_m != a.N * a.tiles_y * a.tiles_x || a.ntiles != a.tiles_m || a.grid < 1 || a.in_sN < 0 || a.in_sH < 0 || a.in_sW < a.unit_C ||
      a.in_sH * a.dw_H * ESZ >= (1ll << 31) || a.in_sN % CE != 0 || a.in_sH % CE != 0 || a.in_sW % CE != 0 || ((uintptr_t)a.in & 15) || a.out_sP % CE != 0 || a.out_sN % CE != 0 ||
      a.out_sP < (a.ileave ? 2 : 1) * a.K || (a.ileave && !a.res))
    return (int)hipErrorInvalidValue;
  const int lds = (int)unit_lds_bytes(a.th, a.tw, s, a.unit_C, a.C, ESZ);
  if (lds > 160 * 1024) return (int)hipErrorInvalidValue;
  static std::atomic<bool> raised{false};
  const hipError_t e = raise_lds_limit(unit_kernel<T>, raised);
  if (e != hipSuccess) return (int)e;
  ConvArgs b = a;
  b.set_quotients();
  if (!b.q_c || !b.q_k) return (int)hipErrorInvalidValue;
  hipLaunchKernelGGL((unit_kernel<T>), dim3(a.grid < a.ntiles ? a.grid : a.ntiles), dim3(UN_NT), lds, st, b);
  return (int)hipGetLastError();
}

int launch_unit(const ConvArgs& a, int dtype, void* stream) {
  return dtype == DT_BF16 ? launch_unit_t<bf16_t>(a, (hipStream_t)stream) : launch_unit_t<float>(a, (hipStream_t)stream);
}

}  // namespace xenos
