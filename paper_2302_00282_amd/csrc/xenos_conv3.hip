// gfx950 (CDNA4) kernels of dense 3x3 / stride 1 / pad 1 convolution chains whose weights do not pass through LDS:
//
//  conv3x3_frag_kernel   bf16, weights from the cache straight into the registers that the MFMAs read: a workgroup of four wavefronts owns a TH x TW block
//                        of output pixels of one image; the input patch of a chunk of 32 channels lies in LDS, every wavefront multiplies all
//                        (or half) of its pixels by 32 output channels of its own.
//  conv3x3_first_kernel  a first layer of at most four channels with its 2x2 pooling on the vector unit, the weights in scalar registers.
#include "device_common.h"

namespace xenos {

typedef __attribute__((ext_vector_type(4))) float acc4_t;

enum { CF_RELU = 1, CF_RES = 2, CF_MAX = 4, CF_RAW = 8 };   // (CF_RAW: fp32 sums [pixel][channel] for the pass that finishes the chain)
struct Frag3Args {
  const void* in; const void* w; const float* scale; const float* shift; const void* res; void* out; const uint16_t* tab;
  uint32_t items, tiles_n, m_tn, tiles_sp, m_sp, tiles_x, m_tx;   // work items, channel tiles, tiles of an image and of a row of it, multipliers
  int32_t nchunks, H, W, K, th, tw, pw; float r_pw;               // chunks of 32 channels; tile; row pitch of the patch in pixels
  uint32_t sN, sH, sW, out_sN, out_sH, out_sP, res_sN, res_sH, res_sP;   // bytes
  int32_t flags;
};

// a value and that of the lane with the lowest bit of its number flipped, or of the lane that mirrors it among eight (two wait states: see quad_max)
template <bool MIRROR>
__device__ __forceinline__ float dpp_max(float v) {
  float r;
  if (MIRROR) asm("s_nop 1\n\tv_max_f32_dpp %0, %1, %1 row_half_mirror row_mask:0xf bank_mask:0xf" : "=v"(r) : "v"(v));
  else asm("s_nop 1\n\tv_max_f32_dpp %0, %1, %1 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf" : "=v"(r) : "v"(v));
  return r;
}
template <bool MIRROR>
__device__ __forceinline__ float dpp_add(float v) {
  float r;
  if (MIRROR) asm("s_nop 1\n\tv_add_f32_dpp %0, %1, %1 row_half_mirror row_mask:0xf bank_mask:0xf" : "=v"(r) : "v"(v));
  else asm("s_nop 1\n\tv_add_f32_dpp %0, %1, %1 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf" : "=v"(r) : "v"(v));
  return r;
}

// Behind which of a chunk's 9 PB fragments a part of the next chunk's patch is requested, and written to LDS
template <int PB, int HALF>
__device__ constexpr int patch_load_at(int it) { return PB > 7 ? (it < HALF ? 2 + 4 * it : 4 * PB + 4 * (it - HALF) + 2) : PB + 2 + 3 * it; }
template <int PB, int HALF>
__device__ constexpr int patch_store_at(int it) { return PB > 7 ? (it < HALF ? 4 * PB + 4 * it : 8 * PB + 4 * (it - HALF)) : 7 * PB + 2 * it; }

// What bounds conv3x3_kernel on these layers is LDS and the barrier of every tap: a tap's weights are written to LDS and read by eight wavefronts, and
// 256 x 128 tiles leave 16 to 19 % of the units' rounds empty.  Here the weights are packed in the order a wavefront loads them and go from the L2
// into the registers that the MFMA reads, two to eight taps ahead: nothing but the pixels passes through LDS, a barrier comes once in nine taps, and
// a workgroup of four wavefronts needs less than half a unit, so that two of them, each at its own place in its own tile, hide one another's epilogues
// and latencies.  A wavefront's 13 blocks of 16 pixels are 14 x 14: the maps of the usual networks are whole numbers of that, 56x56 256 channels at batch
// 32 exactly four tiles a unit, 28x28 512 channels two.  A fragment of 16 pixels (1 KB of LDS) feeds two MFMAs of 16 channels each, which asks for half of what
// LDS can read; 16 x 16 x 32 MFMAs take 18.3 cycles each in this pattern and less power than 32 x 32 x 16 (1820 against 1715 TFLOP/s on random operands).
// Rows are a pitch of five 16-byte slots apart, an odd number, so that a tap is an added offset.  Requests lie between pairs of MFMAs one at a time: two
// in a row hold a wavefront up (43 cycles a tap).
// VGG-16 batch 32: 128 channels 112x112 114 -> 98 us, 256 56x56 115 -> 88 (1340 TFLOP/s), 512 28x28 108 -> 85 (1390), 512 14x14 38 -> 29.5; by the counters MFMA
// pipes are 57 to 66 % busy in the first three at 2.1 to 2.2 GHz, 38 in the last, and 8 to 30 % of the LDS cycles are bank conflicts (most in the pooled forms).
// A workgroup alone on its unit takes 2950 cycles for a chunk of 126 MFMAs: without its weight requests 2600, without its fragment reads 2750.  Three patch
// buffers with the barrier in the middle of a chunk and fragments that run on across chunks took 1 to 10 % longer (they spill, or the barrier waits for more
// reads), fragments nine ahead instead of six the same.
// PB blocks of 16 pixels per wavefront; the four wavefronts are WP groups of pixels x KS shares of the reduction x groups of 32 channels.
template <int PB, int WP, int KS, bool ZIG>
__global__ __launch_bounds__(NT, 2) void conv3x3_frag_kernel(const Frag3Args a) {
  FETCH_ARGS(Frag3Args);
  constexpr int WC = 4 / (WP * KS), BN = 32 * WC, ROWS = WP * PB * 16, LT = NT / KS;   // (LT threads load the patch of a share)
  constexpr int A_IT = frag3_positions(PB, WP) * 4 / LT, AB = frag3_positions(PB, WP) * kFrag3Pitch, RPI = LT / 4;
  constexpr int WS = PB > 7 ? 3 : 9;                               // taps whose weights are in registers or on their way
  constexpr int FD = 6;                                            // fragments of pixels on their way from LDS
  constexpr int B0 = 1, B1 = PB > 4 ? 4 : 3;
  constexpr int HALF = PB > 7 ? (A_IT + 1) / 2 : A_IT;             // the patch of the next chunk travels in two parts, or as a whole
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wc = wave % WC, wp = wave / WC % WP, ks = wave / (WC * WP), row = lane & 15, kg = lane >> 4;
  const int lt = tid - ks * LT;
  unsigned char* const s_in = smem + ks * 2 * AB;                  // this share's two patch buffers
  uint32_t* s_tab = (uint32_t*)(smem + KS * 2 * AB);
  unsigned char* const s_part = smem + KS * 2 * AB + ROWS * 4;     // sums handed from share to share

  // ---- this workgroup's items: an XCD owns a contiguous range of them, (pixel tile, channel tile) with the channel tile fastest
  const uint32_t G = gridDim.x, nx = G >= NUM_XCD ? NUM_XCD : G;
  const uint32_t xcd = G >= NUM_XCD ? blockIdx.x & (NUM_XCD - 1) : blockIdx.x, step = G >= NUM_XCD ? (G - xcd + NUM_XCD - 1) / NUM_XCD : 1;
  const uint32_t end = nx == NUM_XCD ? (xcd + 1) * a.items / NUM_XCD : (xcd + 1) * a.items / nx;
  uint32_t item = (nx == NUM_XCD ? xcd * a.items / NUM_XCD : xcd * a.items / nx) + (G >= NUM_XCD ? blockIdx.x / NUM_XCD : 0);
  if (item >= end) return;                                         // (uniform)
  struct Tile { int tn, n, oy, ox; };
  auto decode = [&](uint32_t t) __attribute__((always_inline)) -> Tile {
    const uint32_t tm = host_quotient(t, a.m_tn), n = host_quotient(tm, a.m_sp), rr = tm - n * a.tiles_sp, ty = host_quotient(rr, a.m_tx);
    return Tile{(int)(t - tm * a.tiles_n), (int)n, (int)ty * a.th, (int)(rr - ty * a.tiles_x) * a.tw};
  };
  Tile cur = decode(item);

  // ---- the input patch: this thread's 16 bytes (chunk lt & 3) of every RPI-th position
  const rsrc_t wa = make_window(a.in, kWindow);
  unsigned poff[A_IT];
  auto patch_addr = [&](const Tile& t) __attribute__((always_inline)) {
    int l = lt;
    asm volatile("" : "+v"(l));                                    // (nothing of it is kept in registers from tile to tile)
#pragma unroll
    for (int it = 0; it < A_IT; ++it) {
      const int p = (l >> 2) + it * RPI, pr = small_quotient(p, a.r_pw), pc = p - pr * a.pw;
      const int ih = t.oy - 1 + pr, iw = t.ox - 1 + pc;
      const bool ok = ((unsigned)ih < (unsigned)a.H) & ((unsigned)iw < (unsigned)a.W) & (pr < a.th + 2) & (pc < a.tw + 2);
      unsigned o = (unsigned)t.n * a.sN + (unsigned)ih * a.sH + (unsigned)iw * a.sW + (l & 3) * 16u;
      asm volatile("" : "+v"(o));                                  // (no branch around it)
      poff[it] = ok ? o : kNoLoad;
    }
  };
  unsigned char* const pdst = s_in + (lt >> 2) * kFrag3Pitch + (lt & 3) * 16;
  u32x4_t pa[HALF];
  auto store_patch = [&](int it, unsigned to) __attribute__((always_inline)) { *(u32x4_t*)(pdst + to + it * RPI * kFrag3Pitch) = pa[it % HALF]; };

  // ---- weights, packed as a wavefront loads them: [32 channels][chunk][tap][block of 16][lane][16 bytes]
  const rsrc_t wb = make_window(a.w, kWindow);
  const unsigned wlane = lane * 16u, wtile = (unsigned)a.nchunks * 9u * 2048u;   // (bytes of 32 channels)
  u32x4_t wr[WS][2];
  auto load_w = [&](int slot, int j, unsigned soff) __attribute__((always_inline)) { wr[slot][j] = load_window(wb, wlane + j * 1024u, soff); };

  // (share ks has chunks ks, ks + KS, ..)
  patch_addr(cur);
  u32x4_t pb[A_IT];
#pragma unroll
  for (int it = 0; it < A_IT; ++it) pb[it] = load_window(wa, poff[it], ks * 64u);
  unsigned wcur = (unsigned)(cur.tn * WC + wc) * wtile + ks * (9u * 2048u);
#pragma unroll
  for (int t = 0; t < WS - 1; ++t) { load_w(t, 0, wcur + t * 2048u); load_w(t, 1, wcur + t * 2048u); }
  // pixel of row r of block b of the tile: (ty << 8) | tx, 0xffff none.  Every lane's LDS address of its pixels' windows
  unsigned abase[PB];
  {
    const unsigned co = (unsigned)(((kg & 1) << 1) | (kg >> 1)) * 16u;
#pragma unroll
    for (int b = 0; b < PB; ++b) {
      const unsigned e = a.tab[(wp * PB + b) * 16 + row];
      abase[b] = (e == 0xffffu ? 0u : ((e >> 8) * (unsigned)a.pw + (e & 255u)) * kFrag3Pitch) + co;
    }
    for (int q = tid; q < ROWS; q += NT) s_tab[q] = a.tab[q];
  }
#pragma unroll
  for (int it = 0; it < A_IT; ++it) *(u32x4_t*)(pdst + it * RPI * kFrag3Pitch) = pb[it];

  acc4_t acc[PB][2];
#pragma unroll
  for (int b = 0; b < PB; ++b) acc[b][0] = acc[b][1] = acc4_t{0.f, 0.f, 0.f, 0.f};
  const unsigned rowstep = (unsigned)a.pw * kFrag3Pitch;
  unsigned flip = AB;                                              // from the buffer that is read to the other one
  unsigned to = AB;                                                // offset of the other one
  int c = ks;
  __syncthreads();

  for (;;) {
    const bool last = c + KS >= a.nchunks;                         // (uniform; the shares have as many chunks each)
    Tile next = cur;
    if (last) {
      if (item + step < end) next = decode(item + step);           // (behind the last item: loads that nobody reads)
      patch_addr(next);
    }
    const unsigned pnext = (unsigned)(last ? ks : c + KS) * 64u;
    const unsigned wnext = last ? (unsigned)(next.tn * WC + wc) * wtile + ks * (9u * 2048u) : wcur + KS * 9u * 2048u;
    u32x4_t fa[FD + 1];
    auto fetch = [&](int q) __attribute__((always_inline)) {       // q-th of the chunk's 9 PB fragments
      const int b = q % PB, tap = q / PB;
      if (tap == 3 || tap == 6) abase[b] += rowstep;
      fa[q % (FD + 1)] = *(const u32x4_t*)(s_in + abase[b] + (tap % 3) * kFrag3Pitch);
    };
#pragma unroll
    for (int q = 0; q < FD; ++q) fetch(q);
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
#pragma unroll
      for (int b = 0; b < PB; ++b) {
        const int q = tap * PB + b;
        if (q + FD < 9 * PB) fetch(q + FD);
        // (accumulator rows = channels, columns = pixels)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[b][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, wr[tap % WS][j]), __builtin_bit_cast(bf16x8_t, fa[q % (FD + 1)]), acc[b][j], 0, 0, 0);
        // one request to memory or write to LDS between two pairs of MFMAs: two in a row hold the wavefront up
        if (b == B0 || b == B1) {                                  // weights of the tap before are used: the next ones for their registers
          const int t = tap == 0 ? WS - 1 : tap - 1 + WS;
          load_w((tap + WS - 1) % WS, b == B1, t < 9 ? wcur + t * 2048u : wnext + (t - 9) * 2048u);
        }
#pragma unroll
        for (int it = 0; it < A_IT; ++it) {
          if (q == patch_load_at<PB, HALF>(it)) pa[it % HALF] = load_window(wa, poff[it], pnext);
          if (q == patch_store_at<PB, HALF>(it)) store_patch(it, to);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    wcur = wnext;
#pragma unroll
    for (int b = 0; b < PB; ++b) abase[b] += flip - 2 * rowstep;
    flip = 0u - flip;
    to = AB - to;
    __syncthreads();
    if (!last) { c += KS; continue; }
    c = ks;

    // ---- the shares' sums: a share finishes half of the blocks and hands the others over.  (Nobody writes here again before every wavefront has
    // passed the barrier behind the next tile's first chunk)
    constexpr int SPLIT = KS > 1 ? (PB + 1) / 2 : PB, UB = 2;   // (UB blocks are finished at a time)
    if constexpr (KS > 1) {
      static_assert(KS == 2 && WP == 1, "two shares");
      f32x4_t* const mine = (f32x4_t*)(s_part + wc * (PB * 2 * 1024)) + lane;
#pragma unroll
      for (int b = 0; b < PB; ++b)
        if ((b < SPLIT) != (ks == 0)) { mine[b * 128] = acc[b][0]; mine[b * 128 + 64] = acc[b][1]; }
      __syncthreads();
#pragma unroll
      for (int b = 0; b < PB; ++b)
        if ((b < SPLIT) == (ks == 0)) { acc[b][0] += mine[b * 128]; acc[b][1] += mine[b * 128 + 64]; }
    }

    if (!ZIG && (a.flags & CF_RAW)) {
      const int k0 = cur.tn * BN + wc * 32 + kg * 8;
      unsigned char* const out = (unsigned char*)a.out + (size_t)(unsigned)cur.n * a.out_sN + (unsigned)k0 * 4u;
#pragma unroll
      for (int b = 0; b < PB; ++b) {
        const uint32_t e = s_tab[(wp * PB + b) * 16 + row];
        const int oy = cur.oy + (int)(e >> 8), ox = cur.ox + (int)(e & 255u);
        if ((b < SPLIT) != (ks == 0) || e == 0xffffu || oy >= a.H || ox >= a.W || k0 >= a.K) continue;
        f32x4_t* const d = (f32x4_t*)(out + ((unsigned)oy * a.out_sH + (unsigned)ox * a.out_sP));
        d[0] = acc[b][0]; d[1] = acc[b][1];
      }
    } else {
    // ---- epilogue: a lane holds channels k0 .. k0 + 7 of a pixel of every block
    int lrow = row, lkg = kg;
    asm volatile("" : "+v"(lrow), "+v"(lkg));
    const int k0 = cur.tn * BN + wc * 32 + lkg * 8;
    float sc[8], sh[8];
#pragma unroll
    for (int e = 0; e < 8; e += 4) {
      *(f32x4_t*)&sc[e] = *(const f32x4_t*)(a.scale + k0 + e);
      *(f32x4_t*)&sh[e] = *(const f32x4_t*)(a.shift + k0 + e);
    }
    const float lo = relu_floor(a.flags & CF_RELU);
    unsigned char* const out = (unsigned char*)a.out + (size_t)(unsigned)cur.n * a.out_sN + (unsigned)k0 * 2u;
    const rsrc_t wres = make_window(a.res, kWindow);
#pragma unroll
    for (int b0 = 0; b0 < PB; b0 += UB) {
      if (KS > 1 && (b0 < SPLIT) != (ks == 0)) continue;           // (uniform)
      uint32_t e4[UB];
      u32x4_t r4[UB];
#pragma unroll
      for (int u = 0; u < UB; ++u)
        if (b0 + u < PB) e4[u] = s_tab[(wp * PB + b0 + u) * 16 + lrow];
      if (!ZIG && (a.flags & CF_RES)) {
#pragma unroll
        for (int u = 0; u < UB; ++u)
          if (b0 + u < PB) {
            const int oy = cur.oy + (int)(e4[u] >> 8), ox = cur.ox + (int)(e4[u] & 255u);
            const bool ok = (e4[u] != 0xffffu) & (oy < a.H) & (ox < a.W) & (k0 < a.K);
            r4[u] = load_window_if(wres, ok, (unsigned)cur.n * a.res_sN + (unsigned)oy * a.res_sH + (unsigned)ox * a.res_sP + (unsigned)k0 * 2u);
          }
      }
#pragma unroll
      for (int u = 0; u < UB; ++u)
        if (b0 + u < PB) {
          const int b = b0 + u, ty = (int)(e4[u] >> 8), tx = (int)(e4[u] & 255u);
          float y[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) y[e] = acc[b][e >> 2][e & 3] * sc[e] + sh[e];
          if (!ZIG && (a.flags & CF_RES)) {
            float r[8];
            Tr<bf16_t>::unpack(r4[u], r);
#pragma unroll
            for (int e = 0; e < 8; ++e) y[e] += r[e];
          }
#pragma unroll
          for (int e = 0; e < 8; ++e) y[e] = fmx_floor(y[e], lo);
          if constexpr (ZIG) {
            if (a.flags & CF_MAX) {
#pragma unroll
              for (int e = 0; e < 8; ++e) y[e] = dpp_max<true>(dpp_max<false>(y[e]));
            } else {
#pragma unroll
              for (int e = 0; e < 8; ++e) y[e] = dpp_add<true>(dpp_add<false>(y[e])) * 0.25f;
            }
          }
          const int oy = cur.oy + ty, ox = cur.ox + tx;
          const bool ok = (e4[u] != 0xffffu) & (oy < a.H) & (ox < a.W) & (k0 < a.K) & (!ZIG || !((ty | tx) & 1));
          const unsigned o = ZIG ? (unsigned)(oy >> 1) * a.out_sH + (unsigned)(ox >> 1) * a.out_sP : (unsigned)oy * a.out_sH + (unsigned)ox * a.out_sP;
          if (ok) *(u32x4_t*)(out + o) = Tr<bf16_t>::pack(y);
        }
      __builtin_amdgcn_sched_barrier(0);
    }
    }
#pragma unroll
    for (int b = 0; b < PB; ++b) acc[b][0] = acc[b][1] = acc4_t{0.f, 0.f, 0.f, 0.f};
    item += step;
    if (item >= end) break;                                        // (uniform)
    cur = next;
  }
}

template <int PB, int WP, int KS, bool ZIG>
static int launch_frag3_inst(const Frag3Args& w, int grid, hipStream_t st) {
  static std::atomic<bool> raised{false};
  const hipError_t e = raise_lds_limit(conv3x3_frag_kernel<PB, WP, KS, ZIG>, raised);
  if (e != hipSuccess) return (int)e;
  hipLaunchKernelGGL((conv3x3_frag_kernel<PB, WP, KS, ZIG>), dim3(grid), dim3(NT), (int)frag3_lds(PB, WP, KS), st, w);
  return (int)hipGetLastError();
}

int launch_frag3(const ConvArgs& a, int dtype, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  const int pb = a.frag3, wp = a.frag3_wp, ks = a.frag3_ks, rows = pb * wp * 16, bn = wp > 0 && ks > 0 ? 128 / (wp * ks) : 0, pw = frag3_pitch(a.tw);
  const bool zig = a.mode == M_ZIGZAG, raw = a.ksplit >= 1;
  // what the kernel assumes, checked again on the host
  if (dtype != DT_BF16 || bn < 32 || a.halo_bn != bn || !frag3_takes(a) || a.C % (32 * ks) != 0 || a.dw_w || a.pair || a.ileave || !a.ktab ||
      (a.mode != M_FLAT && !zig) || (zig && ((a.th | a.tw | a.H | a.W) & 1)) ||
      (raw ? a.ksplit != 1 || zig || a.has_res || !a.part || ((uintptr_t)a.part & 15) || a.part_ld < a.tiles_n * bn || (double)a.M_total * a.part_ld * 4 >= 4294967040.0 || a.M_total != a.N * a.H * a.W
           : !a.vec_out || (a.has_res && (!a.vec_res || !a.res || zig)) || a.out_sK != 1 || a.out_f32) ||
      a.th < 1 || a.tw < 1 || a.th > 255 || a.tw > 255 || a.th * a.tw > rows || (a.th + 2) * pw > frag3_positions(pb, wp) ||
      a.tiles_y != (a.H + a.th - 1) / a.th || a.tiles_x != (a.W + a.tw - 1) / a.tw || a.tiles_m != a.N * a.tiles_y * a.tiles_x ||
      a.tiles_n != (a.K + bn - 1) / bn || (double)a.tiles_m * a.tiles_n >= kHostDiv || a.grid < 1 || a.grid > 0xffff)
    return (int)hipErrorInvalidValue;
  Frag3Args w{};
  w.in = a.in; w.w = a.w; w.scale = a.scale; w.shift = a.shift; w.res = a.has_res ? a.res : nullptr; w.out = a.out; w.tab = (const uint16_t*)a.ktab;
  w.tiles_n = (uint32_t)a.tiles_n; w.m_tn = host_multiplier(w.tiles_n); w.items = (uint32_t)a.tiles_m * w.tiles_n;
  w.tiles_sp = (uint32_t)(a.tiles_y * a.tiles_x); w.m_sp = host_multiplier(w.tiles_sp); w.tiles_x = (uint32_t)a.tiles_x; w.m_tx = host_multiplier(w.tiles_x);
  w.nchunks = a.C / 32; w.H = a.H; w.W = a.W; w.K = a.K; w.th = a.th; w.tw = a.tw; w.pw = pw; w.r_pw = 1.f / (float)pw;
  w.sN = (uint32_t)(a.in_sN * 2); w.sH = (uint32_t)(a.in_sH * 2); w.sW = (uint32_t)(a.in_sW * 2);
  w.out_sN = (uint32_t)(a.out_sN * 2); w.out_sP = (uint32_t)(a.out_sP * 2); w.out_sH = w.out_sP * (uint32_t)(zig ? a.PW : a.OW);
  w.res_sN = (uint32_t)(a.res_sN * 2); w.res_sP = (uint32_t)(a.res_sP * 2); w.res_sH = w.res_sP * (uint32_t)a.OW;
  if (raw) { w.out = a.part; w.out_sP = (uint32_t)a.part_ld * 4; w.out_sH = w.out_sP * (uint32_t)a.OW; w.out_sN = w.out_sH * (uint32_t)a.OH; }
  w.flags = (raw ? CF_RAW : 0) | (a.relu ? CF_RELU : 0) | (a.has_res ? CF_RES : 0) | (zig && a.pool == POOL_MAX ? CF_MAX : 0);
#define XENOS_FRAG3(PB, WP, KS) \
  if (pb == PB && wp == WP && ks == KS) return zig ? launch_frag3_inst<PB, WP, KS, true>(w, a.grid, st) : launch_frag3_inst<PB, WP, KS, false>(w, a.grid, st)
  XENOS_FRAG3(13, 1, 1);
  XENOS_FRAG3(7, 1, 1);
  XENOS_FRAG3(7, 2, 1);
  XENOS_FRAG3(7, 1, 2);
  XENOS_FRAG3(4, 1, 2);
#undef XENOS_FRAG3
  return (int)hipErrorInvalidValue;
}

struct FirstArgs {
  const void* in; const void* w; const float* scale; const float* shift; void* out;
  long long out_sN, out_sP, out_sK;                                // elements
  uint32_t sN, sC, sH, sW, bytes;                                  // bytes; `bytes`: from a channel's first element to behind its last
  int32_t wins, PHW, PW, H, W, blocks, items, groups, wpitch; float r_phw, r_pw;   // pooling windows, blocks of 256 of them, groups of channels, bytes of a channel's weights
  int32_t flags;
};
enum { FF_RELU = 1, FF_MAX = 2, FF_OUT_F32 = 4, FF_VEC = 8 };

// A first layer of few channels in and out (3 -> 16) is neither a matrix product nor bytes: 27 products of a pixel fill a step of 32 or 64 only with an
// import pass in front or a gather of single elements, and 16 channels half a tile.  Here a thread owns a 2x2 pooling window x eight
// channels: the 4 x 4 input pixels of it are in registers, read in the caller's layout; the weights are the wavefront's, in scalar registers, so that a
// product is one instruction; the window is pooled in the thread.  What bounds it is the vector unit's fp32 rate, which without packed instructions is 79 TFLOP/s:
// 25x206x206, 3 -> 16 channels, 0.92 GFLOP, 155 us on conv_kernel behind an import pass -> 21.5 (12 at that rate), 32x256x256 296 -> 35.4.  The products of bf16 numbers are
// exact in fp32, sums are fp32 as the MFMAs' are.
template <typename T, typename TIN, int C>
__global__ __launch_bounds__(NT) void conv3x3_first_kernel(const FirstArgs a) {
  FETCH_ARGS(FirstArgs);
  typedef const __attribute__((address_space(4))) uint32_t* scalar_ptr;
  typedef const __attribute__((address_space(4))) float* scalar_f32;
  // the groups of a block behind one another on one XCD, whose L2 then has the input
  for (int item = (int)blockIdx.x; item < a.items; item += (int)gridDim.x) {
    const int q = item >> 3, qb = uniform_div(q, a.groups), block = qb * 8 + (item & 7), k0 = (q - qb * a.groups) * kFirstChannels;
    if (block >= a.blocks) continue;
    const int win = block * NT + (int)threadIdx.x, w0 = win < a.wins ? win : 0;
    const int n = any_quotient(w0, a.PHW, a.r_phw), p = w0 - n * a.PHW, ph = any_quotient(p, a.PW, a.r_pw), pw = p - ph * a.PW;
    constexpr unsigned OUTSIDE = 1u << 30;                           // (plus any offset inside: beyond the window)
    unsigned ro[4], co[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int y = 2 * ph - 1 + i, x = 2 * pw - 1 + i;
      ro[i] = (unsigned)y < (unsigned)a.H ? (unsigned)n * a.sN + (unsigned)y * a.sH : OUTSIDE;
      co[i] = (unsigned)x < (unsigned)a.W ? (unsigned)x * a.sW : OUTSIDE;
    }
    float x[C][4][4];
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const rsrc_t win_c = make_window((const unsigned char*)a.in + (size_t)c * a.sC, a.bytes);
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          if constexpr (sizeof(TIN) == 4) {
            x[c][r][s] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(win_c, (int)(ro[r] + co[s]), 0, 0));
            if constexpr (sizeof(T) == 2) x[c][r][s] = (float)(__bf16)x[c][r][s];
          } else {
            x[c][r][s] = __uint_as_float((uint32_t)__builtin_amdgcn_raw_buffer_load_b16(win_c, (int)(ro[r] + co[s]), 0, 0) << 16);
          }
        }
    }
    const float lo = a.flags & FF_RELU ? 0.f : __uint_as_float(0x7fc00000u);
    const bool pmax = a.flags & FF_MAX;
    float y[kFirstChannels];
#pragma unroll
    for (int k = 0; k < kFirstChannels; ++k) {
      const scalar_ptr wk = (scalar_ptr)((uintptr_t)a.w + (size_t)(k0 + k) * (unsigned)a.wpitch);
      float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int c = 0; c < C; ++c) {
          const int e = t * C + c, r = t / 3, s = t % 3;
          float w;
          if constexpr (sizeof(T) == 4) w = __uint_as_float(wk[e]);
          else w = __uint_as_float(e & 1 ? wk[e / 2] & 0xffff0000u : wk[e / 2] << 16);
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[j] = fmaf(x[c][r + j / 2][s + j % 2], w, acc[j]);
        }
      const float sc = ((scalar_f32)(uintptr_t)a.scale)[k0 + k], sh = ((scalar_f32)(uintptr_t)a.shift)[k0 + k];
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[j] = fmaxf(fmaf(acc[j], sc, sh), lo);
      y[k] = pmax ? fmaxf(fmaxf(acc[0], acc[1]), fmaxf(acc[2], acc[3])) : ((acc[0] + acc[1]) + (acc[2] + acc[3])) * 0.25f;
    }
    if (win >= a.wins) continue;
    const long long o = (long long)n * a.out_sN + (long long)p * a.out_sP + (long long)k0 * a.out_sK;
    if (sizeof(T) == 2 && !(a.flags & FF_OUT_F32)) {
      bf16_t* out = (bf16_t*)a.out + o;
      if (a.flags & FF_VEC) {
        *(u32x4_t*)out = u32x4_t{f2bf2(y[0], y[1]), f2bf2(y[2], y[3]), f2bf2(y[4], y[5]), f2bf2(y[6], y[7])};
      } else {
#pragma unroll
        for (int k = 0; k < kFirstChannels; ++k) ((uint16_t*)out)[k * a.out_sK] = f2bf(y[k]);
      }
    } else {
      float* out = (float*)a.out + o;
      if (a.flags & FF_VEC) {
        *(f32x4_t*)out = f32x4_t{y[0], y[1], y[2], y[3]};
        *(f32x4_t*)(out + 4) = f32x4_t{y[4], y[5], y[6], y[7]};
      } else {
#pragma unroll
        for (int k = 0; k < kFirstChannels; ++k) out[k * a.out_sK] = y[k];
      }
    }
  }
}

template <typename T, typename TIN>
static int launch_first_t(const FirstArgs& w, int C, int grid, hipStream_t st) {
  switch (C) {
    case 1: hipLaunchKernelGGL((conv3x3_first_kernel<T, TIN, 1>), dim3(grid), dim3(NT), 0, st, w); break;
    case 2: hipLaunchKernelGGL((conv3x3_first_kernel<T, TIN, 2>), dim3(grid), dim3(NT), 0, st, w); break;
    case 3: hipLaunchKernelGGL((conv3x3_first_kernel<T, TIN, 3>), dim3(grid), dim3(NT), 0, st, w); break;
    case 4: hipLaunchKernelGGL((conv3x3_first_kernel<T, TIN, 4>), dim3(grid), dim3(NT), 0, st, w); break;
    default: return (int)hipErrorInvalidValue;
  }
  return (int)hipGetLastError();
}

int launch_first(const ConvArgs& a, int dtype, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  const int esz = dtype == DT_BF16 ? 2 : 4, isz = a.in_f32 ? 4 : esz, osz = a.out_f32 ? 4 : esz;
  const long long wins = (long long)a.N * a.PH * a.PW, blocks = (wins + NT - 1) / NT, groups = a.K / kFirstChannels;
  const long long bytes = ((a.N - 1) * a.in_sN + (a.H - 1) * a.in_sH + (a.W - 1) * a.in_sW + 1) * isz;
  // what the kernel assumes, checked again on the host
  if (a.C < 1 || a.C > 4 || a.R != 3 || a.S != 3 || a.stride != 1 || a.pad != 1 || a.K < kFirstChannels || a.K % kFirstChannels != 0 || a.mode != M_ZIGZAG || a.pk != 2 || a.ps != 2 ||
      a.pp != 0 || a.OH != a.H || a.OW != a.W || 2 * a.PH > a.H || 2 * a.PW > a.W || a.PH < 1 || a.PW < 1 || a.N < 1 || a.has_res || a.ileave || a.dw_w || a.pair || a.kchunk ||
      a.Kred != 9 * a.C || a.Kred_pad < a.Kred || a.Kred_pad % 8 != 0 || a.in_sN < 0 || a.in_sH < 0 || a.in_sW < 0 || a.pair_sC < 0 || a.pair_sC * isz >= (1ll << 32) || bytes > (1ll << 30) ||
      wins >= (1ll << 30) || (blocks + 7) / 8 * 8 * groups >= (1ll << 30) || a.grid < 1 || a.grid > (blocks + 7) / 8 * 8 * groups || (a.pool != POOL_MAX && a.pool != POOL_AVG))
    return (int)hipErrorInvalidValue;
  FirstArgs w{};
  w.in = a.in; w.w = a.w; w.scale = a.scale; w.shift = a.shift; w.out = a.out;
  w.out_sN = a.out_sN; w.out_sP = a.out_sP; w.out_sK = a.out_sK;
  w.sN = (uint32_t)(a.in_sN * isz); w.sC = (uint32_t)(a.pair_sC * isz); w.sH = (uint32_t)(a.in_sH * isz); w.sW = (uint32_t)(a.in_sW * isz); w.bytes = (uint32_t)bytes;
  w.wins = (int)wins; w.PHW = a.PH * a.PW; w.PW = a.PW; w.H = a.H; w.W = a.W; w.blocks = (int)blocks; w.items = (int)((blocks + 7) / 8 * 8 * groups); w.groups = (int)groups; w.wpitch = a.Kred_pad * esz;
  w.r_phw = 1.f / (float)w.PHW; w.r_pw = 1.f / (float)w.PW;
  const bool vec = a.out_sK == 1 && ((uintptr_t)a.out & 15) == 0 && a.out_sN * osz % 16 == 0 && a.out_sP * osz % 16 == 0;
  w.flags = (a.relu ? FF_RELU : 0) | (a.pool == POOL_MAX ? FF_MAX : 0) | (osz == 4 ? FF_OUT_F32 : 0) | (vec ? FF_VEC : 0);
  if (dtype != DT_BF16) return launch_first_t<float, float>(w, a.C, a.grid, st);
  return a.in_f32 ? launch_first_t<bf16_t, float>(w, a.C, a.grid, st) : launch_first_t<bf16_t, bf16_t>(w, a.C, a.grid, st);
}

}  // namespace xenos
