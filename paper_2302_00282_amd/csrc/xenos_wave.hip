// gfx950 (CDNA4) kernels of the chains of few pixels (bf16) and of every dense chain (fp32 at link level 3):
//
//  conv_wave_kernel   implicit-GEMM convolution chain (any kernel size and stride) in tiles of 32 pixels x 32 channels (or 64 x 64), the
//                     reduction of a tile shared out over the four wavefronts of its workgroup (wave_gemm.h); scale / shift, shortcut
//                     and ReLU in the sum of the partial tiles, or raw sums for a reduction that is split over workgroups too.
//  pwdw_wave_kernel   pointwise -> depthwise chain in tiles of at most 32 map positions x 32 channels on the same GEMM.
#include "wave_gemm.h"

namespace xenos {

// What the kernel needs, in the order and form it needs it: three lines of the constant cache, read at once, where the general
// arguments are ten and lead to quotients and products before the first address is known (2800 cycles from the arguments to the
// first request of a 64 x 64 tile).  Byte strides in 32 bits, quotients by multipliers made on the host.
enum { WF_RELU = 1, WF_PARTIAL = 2, WF_OUT_F32 = 4 };
struct WaveConvArgs {
  const void* in; const void* w; const float* scale; const float* shift;
  const void* res; void* out;
  uint32_t tiles, nz, m_nz, ks, m_ks;                  // tiles to visit, channel tiles x shares, shares, multipliers of quotients by them
  int32_t nsteps, steps_per_share;
  uint32_t rs, m_rs, S, m_S; float r_C, r_S;          // taps of the kernel, columns of it, reciprocals
  int32_t M, OHW, OW; float r_ohw, r_ow;
  int32_t stride, pad, H, W, C;
  uint32_t sN, sH, sW, wpitch;                         // bytes
  int32_t K, part_ld, flags;                           // WF_*
  uint32_t out_sN, out_sP, res_sN, res_sP;             // bytes
  int32_t stages;
};

// UNI: the tap of a step is the same for all lanes (1x1, or the taps of a channel chunk in consecutive steps); otherwise every 16 bytes of
// a step have a tap of their own (fewer channels than a step, or a ragged number).
// DIRECT = false: the input lies at an address that is no multiple of 16 bytes (a tensor of the caller's); it then passes through registers
template <typename T, int NB, bool UNI, bool DIRECT>
__global__ __launch_bounds__(NT, NB == 1 ? 4 : 2) void conv_wave_kernel(const WaveConvArgs a) {
  FETCH_ARGS(WaveConvArgs);
  using tr = Tr<T>;
  using tile = WaveTile<T, NB>;
  constexpr int CE = tr::CE, BKE = tr::BKE, ESZ = (int)sizeof(T), EDGE = tile::EDGE;
  extern __shared__ __align__(128) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lrow = lane >> 3, lslot = lane & 7;                    // a request is 8 rows of 8 slots
  const int wave_bytes = a.stages * tile::STAGE;
  unsigned char* s_w = smem + wave * wave_bytes;
  // chunk of a row that the lane loads, of rows 0 .. 7 (16 .. 23) and of rows 8 .. 15 (24 .. 31)
  const int ch[2] = {lslot ^ wave_swizzle(lrow), lslot ^ wave_swizzle(8 + lrow)};
  const rsrc_t wa = make_window(a.in, kWindow);

  for (uint32_t t = blockIdx.x; t < a.tiles; t += gridDim.x) {
    // channel tiles and shares first: where their number is a multiple of eight an XCD reads its own part of the weights only
    const uint32_t tm = host_quotient(t, a.m_nz), z0 = t - tm * a.nz, tn = host_quotient(z0, a.m_ks), z = z0 - tn * a.ks;
    const int s_begin = (int)z * a.steps_per_share;
    const int share = a.nsteps - s_begin < a.steps_per_share ? a.nsteps - s_begin : a.steps_per_share;
    const int n = (share - wave + 3) >> 2;                         // this wavefront's steps: wave, wave + 4, ..
    // the lane's pixel row, handed on to the lanes that load it
    int off, yx;
    {
      const int m = (int)tm * EDGE + (lane & (EDGE - 1));
      const int img = small_quotient(m, a.r_ohw), p = m - img * a.OHW, oh = small_quotient(p, a.r_ow), ow = p - oh * a.OW;
      const int ih = m < a.M ? oh * a.stride - a.pad : -0x4000, iw = ow * a.stride - a.pad;
      off = (int)((unsigned)img * a.sN + (unsigned)ih * a.sH + (unsigned)iw * a.sW);
      yx = (int)(((unsigned)ih << 16) | ((unsigned)iw & 0xffffu));
    }
    int aoff[4 * NB], ayx[4 * NB];
#pragma unroll
    for (int j = 0; j < 4 * NB; ++j) {
      aoff[j] = __builtin_amdgcn_ds_bpermute((j * 8 + lrow) * 4, off) + (UNI ? ch[j & 1] * 16 : 0);
      ayx[j] = __builtin_amdgcn_ds_bpermute((j * 8 + lrow) * 4, yx);
    }
    const unsigned woff[2] = {ESZ == 4 ? lane * 16u : lrow * a.wpitch + ch[0] * 16u, lrow * a.wpitch + ch[1] * 16u};
    const rsrc_t wb = make_window((const unsigned char*)a.w + (size_t)tn * (ESZ == 4 ? NB : EDGE) * a.wpitch, kWindow);
    auto request = [&](int i, unsigned char* dst) __attribute__((always_inline)) {
      const uint32_t s = (uint32_t)(s_begin + wave + 4 * i);
      // row and column of the kernel, offset and validity of the two chunks that the lane loads of a row
      int kr[2], kc[2];
      unsigned koff[2];
      bool kok[2];
      if constexpr (UNI) {
        const uint32_t cc = host_quotient(s, a.m_rs), tap = s - cc * a.rs, r = host_quotient(tap, a.m_S), c = tap - r * a.S;
        const unsigned o = r * a.sH + c * a.sW + cc * (unsigned)ROWB;
#pragma unroll
        for (int v = 0; v < 2; ++v) {
          kr[v] = (int)r; kc[v] = (int)c; koff[v] = o;
          kok[v] = ch[v] * CE < a.C - (int)cc * BKE;               // (the padding of a 1x1 reduction)
        }
      } else {
#pragma unroll
        for (int v = 0; v < 2; ++v) {
          const int kk = (int)s * BKE + ch[v] * CE, tap = small_quotient(kk, a.r_C), c = kk - tap * a.C;
          kr[v] = small_quotient(tap, a.r_S); kc[v] = tap - kr[v] * (int)a.S;
          koff[v] = (unsigned)kr[v] * a.sH + (unsigned)kc[v] * a.sW + c * ESZ;
          kok[v] = tap < (int)a.rs;
        }
      }
#pragma unroll
      for (int j = 0; j < 4 * NB; ++j) {
        const int y = (ayx[j] >> 16) + kr[j & 1], x = (int)(short)ayx[j] + kc[j & 1];
        const bool ok = ((unsigned)y < (unsigned)a.H) & ((unsigned)x < (unsigned)a.W) & kok[j & 1];
        unsigned o = ok ? (unsigned)aoff[j] + koff[j & 1] : kNoLoad;
        asm volatile("" : "+v"(o));
        if constexpr (DIRECT) load_to_lds(wa, dst + j * 1024, o, 0);
        else *(u32x4_t*)(dst + j * 1024 + lane * 16) = load_window(wa, o);
      }
      if constexpr (ESZ == 4) {
#pragma unroll
        for (int j = 0; j < 6 * NB; ++j) load_to_lds(wb, dst + (4 * NB + j) * 1024, woff[0], (j / 6) * a.wpitch + (s * 6 + j % 6) * 1024u);
      } else {
#pragma unroll
        for (int j = 0; j < 4 * NB; ++j) load_to_lds(wb, dst + (4 * NB + j) * 1024, woff[j & 1], j * 8 * a.wpitch + s * ROWB);
      }
    };
    tile::begin(n, a.stages, s_w, request);

    // what the epilogue reads: on its way during the reduction.  The thread finishes channels k .. k + 3 of every RS-th pixel row
    constexpr int RS = NT / tile::SLOTS, U = EDGE / RS;
    const int c4 = tid % tile::SLOTS, k = (int)tn * EDGE + c4 * 4, m0 = (int)tm * EDGE + tid / tile::SLOTS;
    f32x4_t sc = {}, sh = {};
    if (!(a.flags & WF_PARTIAL)) {
      sc = *(const f32x4_t*)(a.scale + k);
      sh = *(const f32x4_t*)(a.shift + k);
    }
    constexpr bool EARLY = NB == 1 || ESZ == 2;                    // (64 x 64 tiles in fp32 have no registers for the shortcut)
    u32x4_t res[U];                                                // (as they lie in memory: converted behind the reduction)
#pragma unroll
    for (int u = 0; u < U; ++u) res[u] = u32x4_t{0u, 0u, 0u, 0u};
    auto load_res = [&]() __attribute__((always_inline)) {
      const rsrc_t wr = make_window(a.res, kWindow);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int m = m0 + u * RS, img = small_quotient(m, a.r_ohw), p = m - img * a.OHW;
        unsigned o = ((m < a.M) & (k < a.K)) ? (unsigned)img * a.res_sN + (unsigned)p * a.res_sP + k * ESZ : kNoLoad;
        asm volatile("" : "+v"(o));
        if constexpr (ESZ == 2) {
          const uint2 r = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(wr, (int)o, 0, 0));
          res[u][0] = r.x; res[u][1] = r.y;
        } else {
          res[u] = load_window(wr, o);
        }
      }
    };
    if (EARLY && a.res) load_res();                                // (uniform)
    tile::finish(n, a.stages, s_w, request);
    if (!EARLY && a.res) load_res();
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int m = m0 + u * RS;
      f32x4_t v = tile::sum(smem, wave_bytes, tid / tile::SLOTS + u * RS, c4);
      if (m >= a.M || k >= a.K) continue;
      if constexpr (ESZ == 4) {
        if (!all_finite(v)) {                                      // with the products of the operands themselves
          const int img = small_quotient(m, a.r_ohw), p = m - img * a.OHW, oh = small_quotient(p, a.r_ow), ow = p - oh * a.OW;
          const unsigned char* const px = (const unsigned char*)a.in + (size_t)((unsigned)img * a.sN);
          v = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
          for (int i = s_begin * BKE; i < (s_begin + share) * BKE; ++i) {
            const int s = i / BKE;
            int tap, c;
            if constexpr (UNI) { const int cc = (int)host_quotient((uint32_t)s, a.m_rs); tap = s - cc * (int)a.rs; c = cc * BKE + i % BKE; }
            else { tap = small_quotient(i, a.r_C); c = i - tap * a.C; }
            const int r = small_quotient(tap, a.r_S), y = oh * a.stride - a.pad + r, x = ow * a.stride - a.pad + tap - r * (int)a.S;
            if (c >= a.C || tap >= (int)a.rs || (unsigned)y >= (unsigned)a.H || (unsigned)x >= (unsigned)a.W) continue;
            const float f = *(const float*)(px + ((unsigned)y * a.sH + (unsigned)x * a.sW + (unsigned)c * 4u));
            const unsigned char* const wst = (const unsigned char*)a.w + (size_t)(NB == 1 ? tn : (unsigned)k / 32) * a.wpitch + (size_t)s * (6 * 1024);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = fmaf(f, wave_weight_f32(wst, (k & 31) + e, i % BKE), v[e]);
          }
        }
      }
      if (a.flags & WF_PARTIAL) {
        *(f32x4_t*)((float*)a.out + ((size_t)z * a.M + m) * a.part_ld + k) = v;
        continue;
      }
      v = v * sc + sh;
      if (a.res) {
        if constexpr (ESZ == 2) v += f32x4_t{bf2f((uint16_t)res[u][0]), __uint_as_float(res[u][0] & 0xffff0000u), bf2f((uint16_t)res[u][1]), __uint_as_float(res[u][1] & 0xffff0000u)};
        else v += __builtin_bit_cast(f32x4_t, res[u]);
      }
      if (a.flags & WF_RELU) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = fmx(v[e], 0.f);
      }
      const int img = small_quotient(m, a.r_ohw), p = m - img * a.OHW;
      unsigned char* dst = (unsigned char*)a.out + (size_t)((unsigned)img * a.out_sN + (unsigned)p * a.out_sP);
      if (ESZ == 4 || (a.flags & WF_OUT_F32)) *(f32x4_t*)(dst + k * 4) = v;
      else *(uint2*)(dst + k * 2) = uint2{f2bf2(v[0], v[1]), f2bf2(v[2], v[3])};
    }
    __syncthreads();                                               // the partial tiles are rewritten
  }
}

// ---------------------------------------------------------------------------------------------
// Pointwise -> depthwise on chip (see pwdw_kernel), for maps of few pixels: a workgroup owns TH x TW depthwise output pixels of one image x 32
// channels, whose windows cover at most kWaveRows pixels of the map.  The pointwise GEMM of that block runs as in conv_wave_kernel; the sum of
// the partial tiles applies the pointwise epilogue and writes the block the stencil reads.  A tile is few outputs
// (8 on a 14x14 map, of 24 to 30 positions), so that the units share the stencil, which is bound by vector instructions.  pwdw_kernel has 16 to 32
// workgroups on such a map; a 64 x 64 chunk there takes 2300 cycles of index arithmetic, 690 per step and 3100 for a stencil of 49 pixels x
// 64 channels.  MobileNet batch 1: bf16 88.0 -> 77.0 us (512 channels 14x14 6.6 -> 5.2), fp32 152.7 -> 100.6.  With 64 positions a tile 79.7
// and 101.9.
// ---------------------------------------------------------------------------------------------
struct WavePwDwArgs {
  const void* in; const void* w; const float* scale; const float* shift;
  const void* dw_w; const float* dw_scale; const float* dw_shift; void* out;
  uint32_t tiles, nh, m_nh, tiles_sp, m_sp, tiles_x, m_tx;   // tiles to visit, 32-channel parts, tiles of an image, tiles of a row, multipliers
  int32_t nsteps, C, K, H, W, OH, OW, th, tw; float r_tw;
  uint32_t sN, sH, sW, wpitch, out_sN, out_sP;         // bytes
  int32_t stride, flags, stages;
};
enum { WF_DW_RELU = 8 };

template <typename T, bool DIRECT>
__global__ __launch_bounds__(NT, 2) void pwdw_wave_kernel(const WavePwDwArgs a) {
  FETCH_ARGS(WavePwDwArgs);
  using tr = Tr<T>;
  using tile = WaveTile<T, 1>;
  constexpr int CE = tr::CE, BKE = tr::BKE, ESZ = (int)sizeof(T), MP = wave_mid_pitch(ESZ), CG = 32 / CE;
  extern __shared__ __align__(128) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lrow = lane >> 3, lslot = lane & 7;
  const int wave_bytes = a.stages * tile::STAGE;
  unsigned char* s_w = smem + wave * wave_bytes;
  unsigned char* s_mid = smem + 4 * wave_bytes;                    // [block position][32 channels]
  const int ch[2] = {lslot ^ wave_swizzle(lrow), lslot ^ wave_swizzle(8 + lrow)};
  const rsrc_t wa = make_window(a.in, kWindow);
  const int s = a.stride, PH = (a.th - 1) * s + 3, PWd = (a.tw - 1) * s + 3;

  for (uint32_t t = blockIdx.x; t < a.tiles; t += gridDim.x) {
    const uint32_t tm = host_quotient(t, a.m_nh), nh = t - tm * a.nh, n = host_quotient(tm, a.m_sp), rr = tm - n * a.tiles_sp, ty = host_quotient(rr, a.m_tx), tx = rr - ty * a.tiles_x;
    const int oy0 = (int)ty * a.th, ox0 = (int)tx * a.tw;          // first depthwise output pixel of the tile
    const int iy0 = oy0 * s - 1, ix0 = ox0 * s - 1;                // map position of block position (0, 0)
    const int y_lo = max(iy0, 0), y_hi = min(iy0 + PH, a.H), x_lo = max(ix0, 0), x_hi = min(ix0 + PWd, a.W);
    const int wv = x_hi - x_lo, npos = (y_hi - y_lo) * wv;         // the part of the block inside the map
    const float r_wv = __builtin_amdgcn_rcpf((float)wv);
    unsigned aoff[4];
    {
      const int m = lane & 31, py = small_quotient(m, r_wv), px = m - py * wv;
      const unsigned off = m < npos ? n * a.sN + (unsigned)(y_lo + py) * a.sH + (unsigned)(x_lo + px) * a.sW : kNoLoad;
#pragma unroll
      for (int j = 0; j < 4; ++j) aoff[j] = (unsigned)__builtin_amdgcn_ds_bpermute((j * 8 + lrow) * 4, (int)off);
    }
    const unsigned woff[2] = {ESZ == 4 ? lane * 16u : lrow * a.wpitch + ch[0] * 16u, lrow * a.wpitch + ch[1] * 16u};
    const rsrc_t wb = make_window((const unsigned char*)a.w + (size_t)nh * (ESZ == 4 ? 1 : 32) * a.wpitch, kWindow);
    auto request = [&](int i, unsigned char* dst) __attribute__((always_inline)) {
      const uint32_t st = (uint32_t)(wave + 4 * i);
      const int left = a.C - (int)st * BKE;                        // (the padding of the reduction)
      if constexpr (ESZ == 4) {
#pragma unroll
        for (int j = 0; j < 6; ++j) load_to_lds(wb, dst + 4096 + j * 1024, woff[0], (st * 6 + j) * 1024u);
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) load_to_lds(wb, dst + 4096 + j * 1024, woff[j & 1], j * 8 * a.wpitch + st * ROWB);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        unsigned o = ((aoff[j] != kNoLoad) & (ch[j & 1] * CE < left)) ? aoff[j] + ch[j & 1] * 16u + st * ROWB : kNoLoad;
        asm volatile("" : "+v"(o));
        if constexpr (DIRECT) load_to_lds(wa, dst + j * 1024, o, 0);
        else *(u32x4_t*)(dst + j * 1024 + lane * 16) = load_window(wa, o);
      }
    };
    const int n_w = (a.nsteps - wave + 3) >> 2;
    tile::begin(n_w, a.stages, s_w, request);

    // what the epilogues read: on its way during the reduction.  In the sum the thread finishes four channels of a position, in the stencil
    // 16 bytes of channels of a pixel
    const int c4 = (tid & 7) * 4, cg = tid % CG, k0 = (int)nh * 32 + cg * CE;
    const bool kok = k0 < a.K;
    const f32x4_t psc = *(const f32x4_t*)(a.scale + nh * 32 + c4), psh = *(const f32x4_t*)(a.shift + nh * 32 + c4);
    u32x4_t dww[9];
#pragma unroll
    for (int t9 = 0; t9 < 9; ++t9) dww[t9] = *(const u32x4_t*)((const T*)a.dw_w + t9 * a.K + (kok ? k0 : 0));
    float dsc[CE], dsh[CE];
#pragma unroll
    for (int e = 0; e < CE; e += 4) {
      *(f32x4_t*)&dsc[e] = *(const f32x4_t*)(a.dw_scale + (kok ? k0 : 0) + e);
      *(f32x4_t*)&dsh[e] = *(const f32x4_t*)(a.dw_shift + (kok ? k0 : 0) + e);
    }
    if (npos < PH * PWd) {                                         // the zero padding of the depthwise convolution
      const u32x4_t z = {0u, 0u, 0u, 0u};
      for (int i = tid; i < PH * PWd * (MP / 16); i += NT) *(u32x4_t*)(s_mid + i * 16) = z;
    }
    tile::finish(n_w, a.stages, s_w, request);
    __syncthreads();
    if (const int m = tid >> 3; m < npos) {
      const int py = small_quotient(m, r_wv), px_ = m - py * wv;
      f32x4_t v = tile::sum(smem, wave_bytes, m, tid & 7);
      if constexpr (ESZ == 4) {
        if (!all_finite(v)) {                                      // with the products of the operands themselves
          const unsigned char* const px = (const unsigned char*)a.in + (size_t)(n * a.sN + (unsigned)(y_lo + py) * a.sH + (unsigned)(x_lo + px_) * a.sW);
          v = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
          for (int i = 0; i < a.C; ++i) {
            const float f = *(const float*)(px + (unsigned)i * 4u);
            const unsigned char* const wst = (const unsigned char*)a.w + (size_t)nh * a.wpitch + (size_t)(i / BKE) * (6 * 1024);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = fmaf(f, wave_weight_f32(wst, c4 + e, i % BKE), v[e]);
          }
        }
      }
      v = v * psc + psh;
      const float lo = relu_floor(a.flags & WF_RELU);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = fmx_floor(v[e], lo);
      unsigned char* dst = s_mid + ((y_lo + py - iy0) * PWd + (x_lo + px_ - ix0)) * MP + c4 * ESZ;
      if constexpr (ESZ == 2) *(uint2*)dst = uint2{f2bf2(v[0], v[1]), f2bf2(v[2], v[3])};
      else *(f32x4_t*)dst = v;
    }
    __syncthreads();                                               // the block is complete

    // ---- depthwise chain out of the block
    if (kok) {
      for (int q = tid / CG; q < a.th * a.tw; q += NT / CG) {
        const int qy = small_quotient(q, a.r_tw), qx = q - qy * a.tw, oy = oy0 + qy, ox = ox0 + qx;
        if (oy >= a.OH || ox >= a.OW) continue;
        const unsigned char* src = s_mid + ((qy * s) * PWd + qx * s) * MP + cg * 16;
        u32x4_t xr[9];
#pragma unroll
        for (int t9 = 0; t9 < 9; ++t9) xr[t9] = *(const u32x4_t*)(src + ((t9 / 3) * PWd + t9 % 3) * MP);
        __builtin_amdgcn_sched_barrier(0);
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
        const float lo = relu_floor(a.flags & WF_DW_RELU);
#pragma unroll
        for (int e = 0; e < CE; ++e) d[e] = fmx_floor(d[e] * dsc[e] + dsh[e], lo);
        *(u32x4_t*)((unsigned char*)a.out + (size_t)(n * a.out_sN + (unsigned)(oy * a.OW + ox) * a.out_sP + (unsigned)k0 * ESZ)) = tr::pack(d);
      }
    }
    __syncthreads();                                               // the partial tiles and the block are rewritten
  }
}

size_t conv_wave_lds(int edge, int stages, int esz) { return (size_t)4 * stages * (esz == 4 ? edge / 32 * kWaveStageF32 : 2 * edge * ROWB); }

// Steps of a wavefront that are on their way at a time: up to four where a unit has one workgroup, two where it has two, one where it has
// more, which then hide each other's latency (3x3 layers in bf16, four in a row: 128 channels 28x28 batch 4, 392 tiles, four 36.8 us, two
// 25.9; 256 channels 14x14 batch 16, 784 tiles, two 60.8, one 56.2; 400 tiles of 144 steps, two 51.8, one 58.5)
// (64 x 64 tiles: a stage is 64 KB.  256 channels 14x14, 196 tiles, one 49.9, two 47.2; 392 tiles, two workgroups to a unit, one 61.9, two 85.3)
// (fp32: a stage is 40 KB, and three of them leave room for the block of a depthwise convolution)
int conv_wave_stages(int edge, int steps, int tiles, int esz) {
  const int n = (steps + 3) / 4, most = edge > kWaveRows ? (tiles <= 256 ? 2 : 1) : tiles <= 256 ? (esz == 4 ? 3 : 4) : tiles <= 512 ? 2 : 1;
  return n < 1 ? 1 : n < most ? n : most;
}

template <typename T, int NB, bool UNI, bool DIRECT>
static int launch_conv_wave_inst(const WaveConvArgs& w, int grid, int lds, hipStream_t st) {
  static std::atomic<bool> raised{false};
  const hipError_t e = raise_lds_limit(conv_wave_kernel<T, NB, UNI, DIRECT>, raised);
  if (e != hipSuccess) return (int)e;
  hipLaunchKernelGGL((conv_wave_kernel<T, NB, UNI, DIRECT>), dim3(std::min((uint32_t)grid, w.tiles)), dim3(NT), lds, st, w);
  return (int)hipGetLastError();
}

template <typename T, int NB>
static int launch_conv_wave_t(const ConvArgs& a, hipStream_t st) {
  constexpr int ESZ = (int)sizeof(T), BKE = Tr<T>::BKE, EDGE = 32 * NB;
  const bool partial = a.ksplit >= 1;
  const int ks = partial ? a.ksplit : 1;
  // what the kernel assumes, checked again on the host
  if (!conv_wave_takes(a, ESZ, EDGE) || a.dw_w || a.pair || a.ileave || a.pool != POOL_NONE || a.tiles_m != (a.M_total + EDGE - 1) / EDGE || a.tiles_n != (a.K + EDGE - 1) / EDGE ||
      (!partial && (a.out_sK != 1 || (a.has_res && (!a.vec_res || !a.res)))) ||
      (partial && (!a.part || a.part_ld < a.tiles_n * EDGE || a.steps_per_split < 1)) || a.grid < 1)
    return (int)hipErrorInvalidValue;
  WaveConvArgs w{};
  w.in = a.in; w.w = a.w; w.scale = a.scale; w.shift = a.shift; w.res = !partial && a.has_res ? a.res : nullptr; w.out = partial ? (void*)a.part : a.out;
  w.nz = (uint32_t)(a.tiles_n * ks); w.m_nz = host_multiplier(w.nz); w.ks = (uint32_t)ks; w.m_ks = host_multiplier(w.ks);
  w.tiles = (uint32_t)a.tiles_m * w.nz;
  w.nsteps = a.Kred_pad / BKE; w.steps_per_share = partial ? a.steps_per_split : w.nsteps;
  w.rs = (uint32_t)(a.R * a.S); w.m_rs = host_multiplier(w.rs); w.S = (uint32_t)a.S; w.m_S = host_multiplier(w.S); w.r_C = 1.f / (float)a.C; w.r_S = 1.f / (float)a.S;
  w.M = a.M_total; w.OHW = a.OH * a.OW; w.OW = a.OW; w.r_ohw = 1.f / (float)w.OHW; w.r_ow = 1.f / (float)w.OW;
  w.stride = a.stride; w.pad = a.pad; w.H = a.H; w.W = a.W; w.C = a.C;
  w.sN = (uint32_t)(a.in_sN * ESZ); w.sH = (uint32_t)(a.in_sH * ESZ); w.sW = (uint32_t)(a.in_sW * ESZ); w.wpitch = (uint32_t)(ESZ == 4 ? a.Kred_pad / BKE * (6 * 1024) : a.Kred_pad * ESZ);   // (of a row, or of a block of 32)
  w.K = a.K; w.part_ld = a.part_ld; w.flags = (a.relu ? WF_RELU : 0) | (partial ? WF_PARTIAL : 0) | (a.out_f32 ? WF_OUT_F32 : 0);
  const int osz = a.out_f32 ? 4 : ESZ;
  w.out_sN = (uint32_t)(a.out_sN * osz); w.out_sP = (uint32_t)(a.out_sP * osz); w.res_sN = (uint32_t)(a.res_sN * ESZ); w.res_sP = (uint32_t)(a.res_sP * ESZ);
  w.stages = conv_wave_stages(EDGE, w.steps_per_share, (int)w.tiles, ESZ);
  const int lds = (int)conv_wave_lds(EDGE, w.stages, ESZ);
  const bool direct = ((uintptr_t)a.in & 15) == 0;
  if (a.R * a.S == 1 || a.kchunk)
    return direct ? launch_conv_wave_inst<T, NB, true, true>(w, a.grid, lds, st) : launch_conv_wave_inst<T, NB, true, false>(w, a.grid, lds, st);
  return direct ? launch_conv_wave_inst<T, NB, false, true>(w, a.grid, lds, st) : launch_conv_wave_inst<T, NB, false, false>(w, a.grid, lds, st);
}

// (fp32 beyond 256 tiles: two stages of 40 KB and the block of the depthwise convolution leave a unit room for one workgroup, one stage for three.  256 channels
// 15x15 batch 3, 480 tiles, a launch of five in a row: with two 7.7 us, MobileNet graph 112.8, with one 5.8 and 103.4; batch 1 224x224 97.4 -> 95.4)
static int pwdw_wave_stages(const ConvArgs& a, int esz) {
  const int tiles = a.tiles_m * ((a.K + 31) / 32);
  if (esz == 4 && tiles > 256) return 1;
  return conv_wave_stages(kWaveRows, a.Kred_pad * esz / ROWB, tiles, esz);
}
size_t pwdw_wave_lds(const ConvArgs& a, int esz) {
  const int s = a.dw_stride;
  return conv_wave_lds(kWaveRows, pwdw_wave_stages(a, esz), esz) + (size_t)((a.th - 1) * s + 3) * ((a.tw - 1) * s + 3) * wave_mid_pitch(esz);
}

template <typename T, bool DIRECT>
static int launch_pwdw_wave_inst(const WavePwDwArgs& w, int grid, int lds, hipStream_t st) {
  static std::atomic<bool> raised{false};
  const hipError_t e = raise_lds_limit(pwdw_wave_kernel<T, DIRECT>, raised);
  if (e != hipSuccess) return (int)e;
  hipLaunchKernelGGL((pwdw_wave_kernel<T, DIRECT>), dim3(std::min((uint32_t)grid, w.tiles)), dim3(NT), lds, st, w);
  return (int)hipGetLastError();
}

template <typename T>
static int launch_pwdw_wave_t(const ConvArgs& a, hipStream_t st) {
  constexpr int ESZ = (int)sizeof(T), BKE = Tr<T>::BKE, CE = Tr<T>::CE;
  const int s = a.dw_stride;
  // what the kernel assumes, checked again on the host: a wrong shape would index outside the LDS block or the tensors
  if (!pwdw_wave_takes(a, ESZ) || a.mode != M_FLAT || a.has_res || a.pool != POOL_NONE || a.ksplit >= 1 || a.ileave || a.kchunk || a.pair || a.dw_panel ||
      a.R != 1 || a.S != 1 || a.stride != 1 || a.pad != 0 || a.C % CE != 0 || a.K % CE != 0 || a.C < CE ||
      a.Kred_pad < (a.C + BKE - 1) / BKE * BKE || a.Kred_pad % BKE != 0 ||
      a.dw_k != 3 || a.dw_pad != 1 || (s != 1 && s != 2) || !a.dw_w || !a.dw_scale || !a.dw_shift || !a.vec_out ||
      a.OH != (a.H + 2 - 3) / s + 1 || a.OW != (a.W + 2 - 3) / s + 1 || a.th < 1 || a.tw < 1 ||
      a.tiles_y != (a.OH + a.th - 1) / a.th || a.tiles_x != (a.OW + a.tw - 1) / a.tw || a.tiles_m != a.N * a.tiles_y * a.tiles_x || a.grid < 1 ||
      a.in_sW < a.C || a.out_sP < a.K || wave_block_positions(a, a.th, a.tw) > kWaveRows)
    return (int)hipErrorInvalidValue;
  WavePwDwArgs w{};
  w.in = a.in; w.w = a.w; w.scale = a.scale; w.shift = a.shift; w.dw_w = a.dw_w; w.dw_scale = a.dw_scale; w.dw_shift = a.dw_shift; w.out = a.out;
  w.nh = (uint32_t)((a.K + 31) / 32); w.m_nh = host_multiplier(w.nh); w.tiles = (uint32_t)a.tiles_m * w.nh;
  w.tiles_sp = (uint32_t)(a.tiles_y * a.tiles_x); w.m_sp = host_multiplier(w.tiles_sp); w.tiles_x = (uint32_t)a.tiles_x; w.m_tx = host_multiplier(w.tiles_x);
  w.nsteps = a.Kred_pad / BKE; w.C = a.C; w.K = a.K; w.H = a.H; w.W = a.W; w.OH = a.OH; w.OW = a.OW; w.th = a.th; w.tw = a.tw; w.r_tw = 1.f / (float)a.tw;
  w.sN = (uint32_t)(a.in_sN * ESZ); w.sH = (uint32_t)(a.in_sH * ESZ); w.sW = (uint32_t)(a.in_sW * ESZ); w.wpitch = (uint32_t)(ESZ == 4 ? a.Kred_pad / BKE * (6 * 1024) : a.Kred_pad * ESZ);   // (of a row, or of a block of 32)
  w.out_sN = (uint32_t)(a.out_sN * ESZ); w.out_sP = (uint32_t)(a.out_sP * ESZ);
  w.stride = s; w.flags = (a.relu ? WF_RELU : 0) | (a.dw_relu ? WF_DW_RELU : 0);
  const int lds = (int)pwdw_wave_lds(a, ESZ);
  w.stages = pwdw_wave_stages(a, ESZ);
  if (lds > kLdsPerUnit) return (int)hipErrorInvalidValue;
  const bool direct = ((uintptr_t)a.in & 15) == 0;
  return direct ? launch_pwdw_wave_inst<T, true>(w, a.grid, lds, st) : launch_pwdw_wave_inst<T, false>(w, a.grid, lds, st);
}

int launch_pwdw_wave(const ConvArgs& a, int dtype, void* stream) {
  return dtype == DT_BF16 ? launch_pwdw_wave_t<bf16_t>(a, (hipStream_t)stream) : launch_pwdw_wave_t<float>(a, (hipStream_t)stream);
}

int launch_conv_wave(const ConvArgs& a, int dtype, int edge, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  if (edge == 64) return dtype == DT_BF16 ? launch_conv_wave_t<bf16_t, 2>(a, st) : launch_conv_wave_t<float, 2>(a, st);
  return dtype == DT_BF16 ? launch_conv_wave_t<bf16_t, 1>(a, st) : launch_conv_wave_t<float, 1>(a, st);
}

}  // namespace xenos
