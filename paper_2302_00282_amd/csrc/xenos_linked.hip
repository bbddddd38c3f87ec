// gfx950 (CDNA4) kernels of the chains whose intermediate tensor stays on chip between two convolutions
// (Table 1, ConvX -> ConvY; Section 2.2 and the last paragraph of Section 4.1):
//
//  pwdw_kernel   pointwise (1x1) convolution chain -> depthwise 3x3 convolution chain.  The pointwise output of a
//                spatial tile plus the one-pixel halo the depthwise windows need lives in LDS only, written there by
//                the GEMM epilogue in the [position][channel] order the depthwise stencil reads.
//  fire_kernel   squeeze 1x1 -> { expand 1x1 || expand 3x3 } -> concat [-> max-pooling] (a Fire module) as one chain: the
//                squeeze tile (+ halo) lives in LDS and is the pixel operand of both expand GEMMs.
#include "device_common.h"

namespace xenos {

// ---------------------------------------------------------------------------------------------
// The 1x1 / stride 1 convolution over all a.C input channels that both kernels below start with, in chunks of 64 pixels x
// 64 output channels.  4 wavefronts as 2 x 2 of 32 pixels x 32 channels; the GEMM is computed transposed, so a lane of
// wavefront (wave_m, wave_n) holds, for pixel row wave_m*32 + l%32, channels k_row0 + wave_n*32 + 8*g + 4*(l/32) + (0..3)
// in acc[4*g .. 4*g+3].  Two LDS stages at s_op (2 * (64 + 64) * LDS_ROW bytes).
// ---------------------------------------------------------------------------------------------
constexpr int PG_BM = 64, PG_BN = 64;
constexpr int PG_STAGES_BYTES = 2 * (PG_BM + PG_BN) * LDS_ROW;

// The GEMMs of ALL chunks of a phase as one sequence of steps (chunk 0 step 0, step 1, ..., chunk 1 step 0, ...): the
// operands of step g + PG_DEPTH are requested from memory when step g is staged, so the memory latency (about 1 us at
// batch 32; timestamps inside the kernels showed it exposed once per chunk, 1.4 us per chunk of a 64-channel layer of
// which 0.3 are work) passes behind the steps before it, across chunk boundaries too.  A ring of PG_DEPTH register sets
// holds the requests in flight, two LDS stages hold the step being multiplied and the next one, one barrier per step.
// `in` is the first pixel that the block reads; pixel(chunk, row) gives the element offset of a row's input pixel from there (-1 = no
// pixel; with nine taps the block's first row and column are the neighbours' where the map has them); epilogue(chunk, acc) receives
// the finished accumulators of a chunk (lane = row wave_m * 32 + l31, channels wave_n * 32 + 8 g + 4 lhalf + 0..3).
// Requests go through buffer windows and are issued on every turn, past the end too (they then read nothing); with a branch around
// them every fourth step waited for all loads in flight, a memory round trip of about 1 us: MobileNet batch 1 102.0 -> 90.1 us, fp32
// 182.2 -> 156.7 (a step of a 512-channel 14x14 layer 0.41 -> 0.28 us, MFMA work 0.06).  Requests past the end are not free in the
// last round, whose loads the caller's next ones queue up behind: 95.2 and 162.1 us with them.
// Ends without a barrier: the caller's next barrier frees the stages.
// TAPS = 9: the convolution is 3x3 / stride 1 / pad 1 instead of 1x1, its weights packed with all taps of a chunk of BKE
// channels in consecutive steps (a.C a multiple of BKE): step s is tap s % 9 of chunk s / 9, the input element of a row
// is its pixel's neighbour at that tap, zero outside the map; coord(chunk, row) gives the pixel's (y << 16) | x.
constexpr int PG_DEPTH = 4;

struct NoCoord { __device__ __forceinline__ int operator()(int, int) const { return 0; } };

template <typename T, int TAPS = 1, typename PixelFn, typename EpiFn, typename CoordFn = NoCoord>
__device__ __forceinline__ void pw_gemm_phase(const ConvArgs& a, const T* in, int k_row0, unsigned char* s_op, int nchunks, PixelFn pixel,
                                              EpiFn epilogue, CoordFn coord = CoordFn()) {
  static_assert(TAPS == 1 || TAPS == 9, "1x1 or 3x3 / pad 1");
  using tr = Tr<T>;
  constexpr int CE = tr::CE, BKE = tr::BKE, ESZ = (int)sizeof(T);
  constexpr int BM = PG_BM, BN = PG_BN, D = PG_DEPTH;
  constexpr int A_IT = BM * CPR / NT, B_IT = BN * CPR / NT;        // 16-byte chunks per thread and step
  static_assert(A_IT >= 1 && B_IT >= 1 && A_IT <= 8 && D % 2 == 0, "loader shapes");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wave_m = wave >> 1, wave_n = wave & 1;
  const int l31 = lane & 31, lhalf = lane >> 5;
  const int nsteps = a.Kred_pad / BKE, G = nchunks * nsteps;
  const int ch = tid % CPR;
  // (what the block reads takes less than 2 GB and 64 rows of weights less than 4: checked by the host.  kFar is beyond the window, and
  // stays so with a step's offset added)
  constexpr unsigned kFar = kBlockWindow;
  const unsigned char* wbase = (const unsigned char*)a.w + (long long)k_row0 * a.Kred_pad * ESZ;
  unsigned woff[B_IT];
#pragma unroll
  for (int it = 0; it < B_IT; ++it) {
    const int idx = tid + it * NT;
    woff[it] = ((unsigned)(idx / CPR) * (unsigned)a.Kred_pad + (idx % CPR) * CE) * ESZ;
  }
  // the chunk and step the next request belongs to, and this thread's input rows of that chunk
  int ld_chunk = -1, ld_step = nsteps - 1;
  unsigned aoff[A_IT];
  int ayx[TAPS == 9 ? A_IT : 1];                                   // TAPS = 9: (y << 16) | x of this thread's rows
  u32x4_t ra[D][A_IT], rb[D][B_IT];
  auto request = [&](int q, int d) __attribute__((always_inline)) {
    const bool more = q < G;                                       // (uniform; the same loads are issued past the end, from empty windows)
    if (more && ++ld_step == nsteps) {
      ld_step = 0;
      ++ld_chunk;
#pragma unroll
      for (int it = 0; it < A_IT; ++it) {
        const int off = pixel(ld_chunk, (tid + it * NT) / CPR);
        aoff[it] = off >= 0 ? (unsigned)(off + ch * CE) * ESZ : kFar;
        if constexpr (TAPS == 9) ayx[it] = coord(ld_chunk, (tid + it * NT) / CPR);
      }
    }
    const rsrc_t wa = make_window(in, more ? kFar : 0), wb = make_window(wbase, more ? kWindow : 0);
    if constexpr (TAPS == 9) {
      const int cch = ld_step / 9, tap = ld_step - cch * 9, dy = tap / 3 - 1, dx = tap - (tap / 3) * 3 - 1;
      const int toff = (dy * (int)a.in_sH + dx * (int)a.in_sW + cch * BKE) * ESZ;
#pragma unroll
      for (int it = 0; it < A_IT; ++it) {
        const int y = (ayx[it] >> 16) + dy, x = (ayx[it] & 0xffff) + dx;
        const bool ok = (aoff[it] < kFar) & ((unsigned)y < (unsigned)a.H) & ((unsigned)x < (unsigned)a.W);
        ra[d][it] = load_window_if(wa, ok, aoff[it] + toff);
      }
    } else {
      const bool kok = ld_step * BKE + ch * CE < a.C;              // channels beyond C are the padding of the reduction
#pragma unroll
      for (int it = 0; it < A_IT; ++it) ra[d][it] = load_window_if(wa, kok, aoff[it] + ld_step * ROWB);
    }
#pragma unroll
    for (int it = 0; it < B_IT; ++it) rb[d][it] = load_window(wb, woff[it], more ? ld_step * ROWB : 0);
  };
  auto store = [&](int stage, int d) __attribute__((always_inline)) {
    unsigned char* sa = s_op + stage * (BM + BN) * LDS_ROW;
    unsigned char* sb = sa + BM * LDS_ROW;
#pragma unroll
    for (int it = 0; it < A_IT; ++it) {
      const int idx = tid + it * NT;
      *(u32x4_t*)(sa + (idx / CPR) * LDS_ROW + (idx % CPR) * 16) = ra[d][it];
    }
#pragma unroll
    for (int it = 0; it < B_IT; ++it) {
      const int idx = tid + it * NT;
      *(u32x4_t*)(sb + (idx / CPR) * LDS_ROW + (idx % CPR) * 16) = rb[d][it];
    }
  };
  f32x16_t acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;
  auto compute = [&](int stage) __attribute__((always_inline)) {
    const unsigned char* sa = s_op + stage * (BM + BN) * LDS_ROW + (wave_m * 32 + l31) * LDS_ROW + lhalf * 16;
    const unsigned char* sb = s_op + stage * (BM + BN) * LDS_ROW + BM * LDS_ROW + (wave_n * 32 + l31) * LDS_ROW + lhalf * 16;
    // (bf16: all fragments of a step requested before its first MFMA: MobileNet batch 1 89.8 -> 88.7 us, SqueezeNet batch 1 80.4 -> 79.8; an
    // fp32 step has sixteen MFMAs to cover the reads, and requested at once they cost 156.5 -> 158.6)
    constexpr int KB = sizeof(T) == 2 ? KG : 1;
#pragma unroll
    for (int k0 = 0; k0 < KG; k0 += KB) {
      u32x4_t fa[KB], fb[KB];
#pragma unroll
      for (int kg = 0; kg < KB; ++kg) { fa[kg] = *(const u32x4_t*)(sa + (k0 + kg) * 32); fb[kg] = *(const u32x4_t*)(sb + (k0 + kg) * 32); }
      if constexpr (KB > 1) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int kg = 0; kg < KB; ++kg) {
        if constexpr (sizeof(T) == 2) {
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, fb[kg]), __builtin_bit_cast(bf16x8_t, fa[kg]), acc, 0, 0, 0);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(fb[kg][e]), __uint_as_float(fa[kg][e]), acc, 0, 0, 0);
        }
      }
    }
  };
#pragma unroll
  for (int d = 0; d < D; ++d) request(d, d);
  int c_chunk = 0, c_step = 0;
  auto multiply = [&](int d) __attribute__((always_inline)) {
    __syncthreads();                                               // the step (and whatever the caller wrote before the phase) is visible
    compute(d & 1);
    if (++c_step == nsteps) {
      epilogue(c_chunk, acc);
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[e] = 0.f;
      c_step = 0;
      ++c_chunk;
    }
  };
  // (no branch around the loads, which would make the next step wait for all of them; the last round requests nothing)
  int g0 = 0;
  for (; g0 + D < G; g0 += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      // stage d % 2 was last read by step g - 2, which every wavefront finished before the barrier of step g - 1
      store(d & 1, d);
      request(g0 + d + D, d);
      multiply(d);
    }
  }
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (d == 0 || g0 + d < G) {                                    // (uniform)
      store(d & 1, d);
      multiply(d);
    }
}

// ---------------------------------------------------------------------------------------------
// Pointwise -> depthwise on chip.
//
// The paper's motivating mismatch (Section 2.2): a producer that writes in one order and a consumer that reads in
// another.  Here the pointwise output never reaches memory at all.  A depthwise convolution works per channel, so
// the pair splits over output channels first (Section 4.2.1) with no redundancy: a workgroup owns a TH x TW block
// of depthwise OUTPUT pixels of one image x 64 channels.  It computes the pointwise chain (GEMM over all input
// channels + scale/shift + ReLU) for the ((TH-1)*s+3) x ((TW-1)*s+3) block of pixels those windows cover, in
// chunks of 64 pixels, straight into an LDS block in the storage type (rounded as a stored tensor would be); block
// positions outside the map stay zero, they are the depthwise padding.  Neighbouring tiles recompute the shared
// border (the paper's halo replication).  Then every thread runs the nine taps of one 16-byte channel group of one
// output pixel out of LDS, applies the depthwise chain's scale/shift/ReLU and stores 16 bytes.
//
// GEMM: 4 wavefronts as 2 x 2 of 32 pixels x 32 channels, operands double-buffered through registers and LDS,
// computed transposed (accumulator rows = channels) so that a lane holds 4 consecutive channels of one pixel.
// ---------------------------------------------------------------------------------------------
constexpr int PD_BM = 64, PD_BN = kPwDwChannels;
__host__ __device__ constexpr int pwdw_mid_pitch(int esz) { return PD_BN * esz + 16; }   // an odd number of 16-byte slots
__host__ __device__ constexpr int pwdw_lds(int positions, int esz) { return positions * pwdw_mid_pitch(esz) + 2 * (PD_BM + PD_BN) * LDS_ROW; }

template <typename T>
__global__ __launch_bounds__(NT, 2) void pwdw_kernel(const ConvArgs a) {
  FETCH_ARGS(ConvArgs);
  using tr = Tr<T>;
  constexpr int CE = tr::CE, ESZ = (int)sizeof(T);
  constexpr int BM = PD_BM, BN = PD_BN;
  constexpr int MP = pwdw_mid_pitch(ESZ);
  constexpr int CG = BN / CE;                                      // 16-byte channel groups of a position
  static_assert(NT % CG == 0 && BM == PG_BM && BN == PG_BN, "loader shapes");
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wave_m = wave >> 1, wave_n = wave & 1;
  const int l31 = lane & 31, lhalf = lane >> 5;

  const int s = a.dw_stride;
  const int PH = (a.th - 1) * s + 3, PWd = (a.tw - 1) * s + 3;      // staged block of the pointwise output
  unsigned char* s_mid = smem;
  unsigned char* s_op = smem + PH * PWd * MP;
  const int tiles_sp = a.tiles_y * a.tiles_x;
  const int cg = tid % CG;
  const SmallDiv by_tw(a.tw);

  for (int t = blockIdx.x; t < a.ntiles; t += gridDim.x) {
    const int tile_n = tile_div(t, a.tiles_m, a.q_tm), tm = t - tile_n * a.tiles_m;  // neighbours share a weight slice
    const int n = tile_div(tm, tiles_sp, a.q_sp), rr = tm - n * tiles_sp, ty = tile_div(rr, a.tiles_x, a.q_tx), tx = rr - ty * a.tiles_x;
    const int oy0 = ty * a.th, ox0 = tx * a.tw;                    // first depthwise output pixel of the tile
    const int iy0 = oy0 * s - 1, ix0 = ox0 * s - 1;                // map position of block position (0, 0)
    const int y_lo = iy0 > 0 ? iy0 : 0, y_hi = iy0 + PH < a.H ? iy0 + PH : a.H;
    const int x_lo = ix0 > 0 ? ix0 : 0, x_hi = ix0 + PWd < a.W ? ix0 + PWd : a.W;
    const int hv = y_hi - y_lo, wv = x_hi - x_lo, npos = hv * wv;   // the part of the block inside the map (never empty)
    const SmallDiv by_wv(wv);

    // this thread's depthwise weights and folded scale / shift: its channel group is the same for all its pixels
    const int k0 = tile_n * BN + cg * CE;
    const bool kok = k0 < a.K;
    u32x4_t dww[9];
#pragma unroll
    for (int t9 = 0; t9 < 9; ++t9) dww[t9] = *(const u32x4_t*)((const T*)a.dw_w + (long long)t9 * a.K + (kok ? k0 : 0));

    float dsc[CE], dsh[CE];
#pragma unroll
    for (int e = 0; e < CE; e += 4) {
      *(f32x4_t*)&dsc[e] = *(const f32x4_t*)(a.dw_scale + (kok ? k0 : 0) + e);
      *(f32x4_t*)&dsh[e] = *(const f32x4_t*)(a.dw_shift + (kok ? k0 : 0) + e);
    }

    if (hv < PH || wv < PWd) {
      // the block overhangs the map: those positions are the zero padding of the depthwise convolution
      const u32x4_t z = {0u, 0u, 0u, 0u};
      for (int i = tid; i < PH * PWd * (MP / 16); i += NT) *(u32x4_t*)(s_mid + i * 16) = z;
    }

    // scale and shift of this lane's channels: the same for every chunk, requested once
    f32x4_t psc[4], psh[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int kk = tile_n * BN + wave_n * 32 + g * 8 + lhalf * 4;
      psc[g] = *(const f32x4_t*)(a.scale + kk);
      psh[g] = *(const f32x4_t*)(a.shift + kk);
    }
    // ---- pointwise GEMM of the block, 64 positions x 64 channels per chunk over all input channels, and the pointwise
    // chain's epilogue into the LDS block: lane = position wave_m*32 + l31, channels wave_n*32 + 8*g + 4*lhalf + (0..3)
    const T* first = (const T*)a.in + (long long)n * a.in_sN + (long long)y_lo * a.in_sH + (long long)x_lo * a.in_sW;
    pw_gemm_phase<T>(a, first, tile_n * BN, s_op, (npos + BM - 1) / BM, [&](int mc, int row) -> int {
      const int m = mc * BM + row;
      if (m >= npos) return -1;
      const int py = by_wv(m), px = m - py * wv;
      return py * (int)a.in_sH + px * (int)a.in_sW;
    }, [&](int mc, const f32x16_t& acc) {
      const int m = mc * BM + wave_m * 32 + l31;
      if (m < npos) {
        const int py = by_wv(m), px = m - py * wv;
        unsigned char* dst = s_mid + ((y_lo + py - iy0) * PWd + (x_lo + px - ix0)) * MP;
        const float lo = relu_floor(a.relu);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int c = wave_n * 32 + g * 8 + lhalf * 4;
          const f32x4_t sc = psc[g], sh = psh[g];
          float y[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) y[e] = fmx_floor(acc[4 * g + e] * sc[e] + sh[e], lo);
          if constexpr (sizeof(T) == 2) {
            uint2 o;
            o.x = f2bf2(y[0], y[1]);
            o.y = f2bf2(y[2], y[3]);
            *(uint2*)(dst + c * 2) = o;
          } else {
            *(f32x4_t*)(dst + c * 4) = f32x4_t{y[0], y[1], y[2], y[3]};
          }
        }
      }
    });
    __syncthreads();                                               // the block is complete

    // ---- depthwise chain out of the block: one thread = one 16-byte channel group of one output pixel --------
    if (kok) {
      for (int q = tid / CG; q < a.th * a.tw; q += NT / CG) {
        const int qy = by_tw(q), qx = q - qy * a.tw;
        const int oy = oy0 + qy, ox = ox0 + qx;
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
#pragma unroll
        for (int e = 0; e < CE; ++e) {
          const float y = d[e] * dsc[e] + dsh[e];
          d[e] = a.dw_relu ? fmx(y, 0.f) : y;
        }
        *(u32x4_t*)((T*)a.out + (long long)n * a.out_sN + (long long)(oy * a.OW + ox) * a.out_sP + k0) = tr::pack(d);
      }
    }
    __syncthreads();                                               // the block is rewritten by the next tile
  }
}

template <typename T>
static int launch_pwdw_t(const ConvArgs& a, hipStream_t st) {
  constexpr int ESZ = (int)sizeof(T), BKE = Tr<T>::BKE, CE = Tr<T>::CE;
  const int s = a.dw_stride;
  // what the kernel assumes, checked again on the host: a wrong shape would index outside the LDS block or the tensors
  if (a.mode != M_FLAT || a.has_res || a.pool != POOL_NONE || a.ksplit >= 1 || a.ileave || a.kchunk || a.pair || a.dw_panel ||
      a.R != 1 || a.S != 1 || a.stride != 1 || a.pad != 0 || a.C % CE != 0 || a.K % CE != 0 || a.C < CE ||
      a.Kred_pad < (a.C + BKE - 1) / BKE * BKE || a.Kred_pad % BKE != 0 ||
      a.dw_k != 3 || a.dw_pad != 1 || (s != 1 && s != 2) || !a.dw_w || !a.dw_scale || !a.dw_shift || !a.vec_out ||
      a.OH != (a.H + 2 - 3) / s + 1 || a.OW != (a.W + 2 - 3) / s + 1 || a.th < 1 || a.tw < 1 ||
      a.tiles_y != (a.OH + a.th - 1) / a.th || a.tiles_x != (a.OW + a.tw - 1) / a.tw || a.tiles_m != a.N * a.tiles_y * a.tiles_x ||
      a.tiles_n != (a.K + PD_BN - 1) / PD_BN || a.ntiles != a.tiles_m * a.tiles_n || a.grid < 1 ||
      a.in_sN < 0 || a.in_sH < 0 || a.in_sW < a.C || !block_window_fits(a, (a.th - 1) * s + 3, ESZ) || a.out_sP < a.K)
    return (int)hipErrorInvalidValue;
  const int positions = ((a.th - 1) * s + 3) * ((a.tw - 1) * s + 3);
  const int lds = pwdw_lds(positions, ESZ);
  if (positions > kPwDwMaxPositions || lds > 160 * 1024) return (int)hipErrorInvalidValue;
  static std::atomic<bool> raised{false};
  const hipError_t e = raise_lds_limit(pwdw_kernel<T>, raised);
  if (e != hipSuccess) return (int)e;
  ConvArgs b = a;
  b.set_quotients();
  hipLaunchKernelGGL((pwdw_kernel<T>), dim3(a.grid < a.ntiles ? a.grid : a.ntiles), dim3(NT), lds, st, b);
  return (int)hipGetLastError();
}

int launch_pwdw(const ConvArgs& a, int dtype, void* stream) {
  return dtype == DT_BF16 ? launch_pwdw_t<bf16_t>(a, (hipStream_t)stream) : launch_pwdw_t<float>(a, (hipStream_t)stream);
}

size_t pwdw_lds_bytes(int th, int tw, int stride, int esz) {
  return (size_t)pwdw_lds(((th - 1) * stride + 3) * ((tw - 1) * stride + 3), esz);
}

// ---------------------------------------------------------------------------------------------
// Fire module on chip: squeeze 1x1 -> { expand 1x1  ||  expand 3x3 / pad 1 } -> channel concat [-> max-pooling] as ONE
// chain (Table 1, Conv1x1 -> Conv3x3; Section 4.1, last paragraph: the consumer's halo is replicated per tile).
//
// The squeeze output has few channels (16 .. 64) and two readers; kept in LDS it is written once and never reaches
// memory.  A workgroup owns a TH x TW tile of output pixels of one image and a share of the expand channels:
//   phase 1  the squeeze chain (GEMM over all input channels + scale/shift + ReLU) for the (TH+2) x (TW+2) block of
//            pixels the 3x3 windows cover, in chunks of 64 positions, into an LDS block [position][S channels] in the
//            storage type; positions outside the map stay zero (the padding of the 3x3 convolution);
//   phase 2  for each of its 64-channel expand tiles every chunk of 64 pixels runs its 1 or 9 taps as MFMAs whose pixel operand
//            is read from the squeeze block at the tap's offset and whose weight operand lies in the wavefront's registers
//            (bf16; requested from memory behind the squeeze GEMM) or in LDS (fp32: the tile's weights, all taps, copied
//            there once): no barrier inside; the epilogue (scale/shift/ReLU) is per wavefront, staged through a private LDS
//            slice and stored as 16-byte channel groups at the part's channel offset in the concat buffer (Eq. 1: the
//            halves join without a layout pass).
// With a linked 3x3 / stride 2 max-pooling (ceil mode; the planner hoists the pooling over the concat) the tile is PTH x
// PTW pooling windows: the expand results of the (2 PTH + 1) x (2 PTW + 1) pixels they cover are staged per channel tile
// in LDS and one thread per 16-byte channel group of a window takes the maximum.
// Workgroups of different channel shares recompute the squeeze block of their tile.
// ---------------------------------------------------------------------------------------------
__host__ __device__ constexpr int fire_sq_pitch(int S, int esz) { return S * esz + 16; }
__host__ __device__ constexpr int fire_w_pitch(int taps, int S, int esz) { return taps * S * esz + 16; }
__host__ __device__ constexpr int fire_stg_pitch(int esz) { return 32 * esz + 16; }
__host__ __device__ constexpr int fire_cb_pitch(int esz) { return 64 * esz + 16; }
// LDS, fp32: squeeze block | max(GEMM stages, one 3x3 weight tile) | 4 per-wavefront staging slices | pooled form: conv block of
// a channel tile.  bf16: squeeze block | GEMM stages, whose space the staging slices and the conv block take over afterwards.
__host__ __device__ constexpr int fire_lds(int positions, int S, int esz, int pool_positions) {
  return esz == 2 ? positions * fire_sq_pitch(S, esz) + cmax(PG_STAGES_BYTES, 4 * 32 * fire_stg_pitch(esz) + pool_positions * fire_cb_pitch(esz))
                  : positions * fire_sq_pitch(S, esz) + cmax(PG_STAGES_BYTES, 64 * fire_w_pitch(9, S, esz)) + 4 * 32 * fire_stg_pitch(esz) +
                        pool_positions * fire_cb_pitch(esz);
}

// KGS (bf16): S / 16, the MFMA k-groups of a tap.  The weights of a wavefront's 32 expand channels, 1 or 9 taps x KGS fragments
// packed in fragment order, then go from memory straight into registers and stay there for all pixel chunks of the tile: the
// first 1x1 tile's are requested before phase 1 and the first 3x3 tile's behind it, so their latency passes under the GEMMs,
// phase 2 has no barrier (unpooled) and reads only pixel fragments from LDS.  Staged through LDS, a 3x3 tile over 64 channels
// cost a copy of 3.2 us before its first MFMA and twice the fragment reads (SqueezeNet bf16 batch 1 121 -> 94 us, batch 32
// 242 -> 203 us).  The fragments must not be undefined on any path: their registers are then kept over the whole kernel.  With 64
// squeeze channels a 3x3 tile is 144 registers of the 256: the last four of its nine taps are requested behind the 1x1 tiles, whose
// registers they take (the first five cover their latency), and nothing of the lane's addresses is kept from tile to tile.
// Requested all at once, 23 to 36 registers were spilled (modules of 64 squeeze channels 4 to 28 % slower, ones of a pair that
// ends in a 1x1 convolution slower than through LDS).  KGS = 0 (fp32, whose fragments do not fit the registers): the weights of a
// tile are copied to LDS.
template <typename T, bool POOL, int TAPS1, int KGS>
__global__ __launch_bounds__(NT, 2) void fire_kernel(const ConvArgs a) {
  FETCH_ARGS(ConvArgs);
  using tr = Tr<T>;
  constexpr int CE = tr::CE, ESZ = (int)sizeof(T);
  constexpr int STP = fire_stg_pitch(ESZ), CBP = fire_cb_pitch(ESZ);
  constexpr int G = 32 * ESZ / 16;                                 // 16-byte channel groups of a wavefront's 32 channels
  extern __shared__ __align__(16) unsigned char smem[];
  const int wave = (int)threadIdx.x >> 6, wave_m = wave >> 1, wave_n = wave & 1;

  const int S = a.K;                                               // squeeze channels
  const int SQP = fire_sq_pitch(S, ESZ);
  const int kgs = S * ESZ / 32;                                    // MFMA k-groups per tap
  // conv-output pixels of a tile: th x tw, or the block the tile's pooling windows cover
  const int CH = POOL ? (a.pph - 1) * a.ps + a.pk : a.th, CW = POOL ? (a.ppw - 1) * a.ps + a.pk : a.tw;
  // the block of the first convolution's output a tile reads: its pixels, and one ring of halo when a 3x3 part exists
  const int ring = a.fire_E[1] > 0 ? 1 : 0;
  const int PH = CH + 2 * ring, PWd = CW + 2 * ring;
  unsigned char* s_sq = smem;
  unsigned char* s_b = smem + PH * PWd * SQP;
  const int bbytes = 64 * fire_w_pitch(9, S, ESZ);
  unsigned char* s_free = KGS > 0 ? s_b : s_b + (bbytes > PG_STAGES_BYTES ? bbytes : PG_STAGES_BYTES);
  unsigned char* s_stg = s_free + wave * 32 * STP;
  unsigned char* s_cb = s_free + 4 * 32 * STP;                     // POOL: [conv pixel][64 channels]
  const int tiles_sp = a.tiles_y * a.tiles_x;
  const int npix = CH * CW;
  const SmallDiv by_cw(CW), by_ppw(POOL ? a.ppw : 1);

  for (int t = blockIdx.x; t < a.ntiles; t += gridDim.x) {
    // (64 squeeze channels, or 48 with a pooling: what follows from the lane's number is worked out per tile and not kept over all tiles, for whose
    // registers the expand weights have no room)
    int tid = (int)threadIdx.x;
    if constexpr (KGS == 4 || (KGS == 3 && POOL)) asm volatile("" : "+v"(tid));
    const int lane = tid & 63, l31 = lane & 31, lhalf = lane >> 5;
    const int gz = tile_div(t, a.tiles_m, a.q_tm), tm = t - gz * a.tiles_m;   // channel share, spatial tile
    const int n = tile_div(tm, tiles_sp, a.q_sp), rr = tm - n * tiles_sp, ty = tile_div(rr, a.tiles_x, a.q_tx), tx = rr - ty * a.tiles_x;
    // first conv-output pixel of the tile
    const int oy0 = POOL ? ty * a.pph * a.ps - a.pp : ty * a.th, ox0 = POOL ? tx * a.ppw * a.ps - a.pp : tx * a.tw;
    const int iy0 = oy0 - ring, ix0 = ox0 - ring;                  // map position of block position (0, 0)
    const int y_lo = iy0 > 0 ? iy0 : 0, y_hi = iy0 + PH < a.H ? iy0 + PH : a.H;
    const int x_lo = ix0 > 0 ? ix0 : 0, x_hi = ix0 + PWd < a.W ? ix0 + PWd : a.W;
    const int hv = y_hi - y_lo, wv = x_hi - x_lo, npos = hv * wv;   // the part of the block inside the map (never empty)
    const SmallDiv by_wv(wv);

    if (hv < PH || wv < PWd) {
      const u32x4_t z = {0u, 0u, 0u, 0u};
      for (int i = tid; i < PH * PWd * (SQP / 16); i += NT) *(u32x4_t*)(s_sq + i * 16) = z;
    }
    // KGS > 0: this wavefront's weight fragments of the first tile of each part
    u32x4_t w0[KGS > 0 ? KGS : 1];
    auto load_w = [&](int which, int j, auto& w, auto F0, auto F1) __attribute__((always_inline)) {   // fragments F0 .. F1
      constexpr int NF = sizeof(w) / sizeof(u32x4_t);
      if (j * 64 < a.fire_E[which]) {                              // (uniform)
        const u32x4_t* src = (const u32x4_t*)a.fire_w[which] + (j * 2 + wave_n) * NF * 64 + lane;
#pragma unroll
        for (int f = F0(); f < F1(); ++f) w[f] = src[f * 64];
      } else {                                                     // (not left undefined: the registers would be kept over the whole kernel)
#pragma unroll
        for (int f = F0(); f < F1(); ++f) w[f] = u32x4_t{0u, 0u, 0u, 0u};
      }
    };
    constexpr std::integral_constant<int, 0> f_begin;
    constexpr std::integral_constant<int, KGS> f_end1;
    constexpr std::integral_constant<int, 9 * KGS> f_end9;
    constexpr std::integral_constant<int, (KGS == 4 ? 5 : 9) * KGS> f_ahead9;   // of a 3x3 tile: requested before the 1x1 tiles
    // first tile of either part: the 3x3 part's tiles and then the 1x1 part's are dealt to the shares one by one
    const int j_first[2] = {gz >= a.fire_skip ? gz - a.fire_skip : gz - a.fire_skip + a.tiles_n, gz};
    if constexpr (KGS > 0) load_w(0, j_first[0], w0, f_begin, f_end1);

    // ---- phase 1: the squeeze chain of the block, into LDS -------------------------------------------------
    // (scale and shift of this lane's channels are the same for every chunk: requested once)
    f32x4_t qsc[4], qsh[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int c = wave_n * 32 + g * 8 + lhalf * 4;
      qsc[g] = *(const f32x4_t*)(a.scale + (c < S ? c : 0));
      qsh[g] = *(const f32x4_t*)(a.shift + (c < S ? c : 0));
    }
    const int yb = TAPS1 == 9 && y_lo > 0 ? 1 : 0, xb = TAPS1 == 9 && x_lo > 0 ? 1 : 0;   // rows and columns read before the block's
    const T* first = (const T*)a.in + (long long)n * a.in_sN + (long long)(y_lo - yb) * a.in_sH + (long long)(x_lo - xb) * a.in_sW;
    pw_gemm_phase<T, TAPS1>(a, first, 0, s_b, (npos + 63) / 64, [&](int mc, int row) -> int {
      const int m = mc * 64 + row;
      if (m >= npos) return -1;
      const int py = by_wv(m), px = m - py * wv;
      return (yb + py) * (int)a.in_sH + (xb + px) * (int)a.in_sW;
    }, [&](int mc, const f32x16_t& acc) {
      const int m = mc * 64 + wave_m * 32 + l31;
      if (m < npos) {
        const int py = by_wv(m), px = m - py * wv;
        unsigned char* dst = s_sq + ((y_lo + py - iy0) * PWd + (x_lo + px - ix0)) * SQP;
        const float lo = relu_floor(a.relu);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int c = wave_n * 32 + g * 8 + lhalf * 4;
          if (c < S) {
            const f32x4_t sc = qsc[g], sh = qsh[g];
            float y[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) y[e] = fmx_floor(acc[4 * g + e] * sc[e] + sh[e], lo);
            if constexpr (sizeof(T) == 2) {
              uint2 o;
              o.x = f2bf2(y[0], y[1]);
              o.y = f2bf2(y[2], y[3]);
              *(uint2*)(dst + c * 2) = o;
            } else {
              *(f32x4_t*)(dst + c * 4) = f32x4_t{y[0], y[1], y[2], y[3]};
            }
          }
        }
      }
    }, [&](int mc, int row) -> int {
      const int m = mc * 64 + row, mm = m < npos ? m : 0;
      const int py = by_wv(mm), px = mm - py * wv;
      return ((y_lo + py) << 16) | (x_lo + px);
    });
    __syncthreads();                                               // the block is complete, the GEMM stages are free

    // ---- phase 2: this workgroup's expand tiles -----------------------------------------------------------
    // epilogue of a wavefront's 32 pixels x 32 channels of chunk mc of channel tile j
    auto load_affine = [&](int which, int j, f32x4_t* esc, f32x4_t* esh) __attribute__((always_inline)) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int kk = j * 64 + wave_n * 32 + g * 8 + lhalf * 4;
        esc[g] = *(const f32x4_t*)(a.fire_scale[which] + kk);
        esh[g] = *(const f32x4_t*)(a.fire_shift[which] + kk);
      }
    };
    auto tile_epilogue = [&](int which, int j, int mc, const f32x16_t& acc, const f32x4_t* esc, const f32x4_t* esh) __attribute__((always_inline)) {
      const int E = a.fire_E[which];
      const float lo = relu_floor(a.fire_relu[which]);
      // finished values change hands inside the wavefront only
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int c = g * 8 + lhalf * 4;
        const f32x4_t sc = esc[g], sh = esh[g];
        float y[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = fmx_floor(acc[4 * g + e] * sc[e] + sh[e], lo);
        if constexpr (sizeof(T) == 2) {
          uint2 o;
          o.x = f2bf2(y[0], y[1]);
          o.y = f2bf2(y[2], y[3]);
          *(uint2*)(s_stg + l31 * STP + c * 2) = o;
        } else {
          *(u32x4_t*)(s_stg + l31 * STP + c * 4) = u32x4_t{__float_as_uint(y[0]), __float_as_uint(y[1]), __float_as_uint(y[2]), __float_as_uint(y[3])};
        }
      }
#pragma unroll
      for (int u = 0; u < 32 * G / 64; ++u) {
        const int idx = lane + u * 64, r = idx / G, cg = idx - r * G;
        const int mr = mc * 64 + wave_m * 32 + r;
        const int k0 = j * 64 + wave_n * 32 + cg * CE;
        u32x4_t v;
        if constexpr (sizeof(T) == 2) {
          const uint2 lo8 = *(const uint2*)(s_stg + r * STP + cg * 16), hi8 = *(const uint2*)(s_stg + r * STP + cg * 16 + 8);
          v = u32x4_t{lo8.x, lo8.y, hi8.x, hi8.y};
        } else {
          v = *(const u32x4_t*)(s_stg + r * STP + cg * 16);
        }
        if (mr < npix && k0 < E) {
          const int qy = by_cw(mr), qx = mr - qy * CW;
          if constexpr (POOL) {
            *(u32x4_t*)(s_cb + mr * CBP + (wave_n * 32 + cg * CE) * ESZ) = v;
          } else {
            const int oy = oy0 + qy, ox = ox0 + qx;
            if (oy < a.H && ox < a.W)
              *(u32x4_t*)((T*)a.fire_out[which] + (long long)n * a.fire_sN[which] + (long long)(oy * a.W + ox) * a.fire_sP[which] + k0) = v;
          }
        }
      }
    };
    // POOL: the windows of channel tile j out of its conv block
    auto tile_pool = [&](int which, int j) __attribute__((always_inline)) {
      const int E = a.fire_E[which];
      __syncthreads();                                         // the conv block of this channel tile is complete
      // one thread = one 16-byte channel group of one pooling window; windows are clipped to the map (never empty)
      constexpr int CG = 64 / CE;
      for (int idx = tid; idx < a.pph * a.ppw * CG; idx += NT) {
        const int q = idx / CG, cg = idx - q * CG, k0 = j * 64 + cg * CE;
        const int qy = by_ppw(q), qx = q - qy * a.ppw;
        const int gy = ty * a.pph + qy, gx = tx * a.ppw + qx;
        if (gy >= a.PH || gx >= a.PW || k0 >= E) continue;
        float mx[CE];
#pragma unroll
        for (int e = 0; e < CE; ++e) mx[e] = -INFINITY;
        if (a.pk == 3) {
          // all nine reads of the window are issued before the first maximum (elements outside the map read the
          // window's first element, which is inside, once more): as a loop over rows and columns the stage paid one
          // LDS latency per element, 3 of the 21 us of a pooled module's workgroup at batch 32
          u32x4_t wv9[9];
#pragma unroll
          for (int t9 = 0; t9 < 9; ++t9) {
            const int cy = qy * a.ps + t9 / 3, cx = qx * a.ps + t9 % 3;
            const bool in = oy0 + cy < a.H && ox0 + cx < a.W;   // (no padding: windows start inside the map)
            wv9[t9] = *(const u32x4_t*)(s_cb + (in ? cy * CW + cx : qy * a.ps * CW + qx * a.ps) * CBP + cg * 16);
          }
#pragma unroll
          for (int t9 = 0; t9 < 9; ++t9) {
            float x[CE];
            tr::unpack(wv9[t9], x);
#pragma unroll
            for (int e = 0; e < CE; ++e) mx[e] = fmx_raw(mx[e], x[e]);
          }
        } else {
          for (int r = 0; r < a.pk; ++r)
            for (int c = 0; c < a.pk; ++c) {
              const int cy = qy * a.ps + r, cx = qx * a.ps + c;
              const int oy = oy0 + cy, ox = ox0 + cx;
              if (oy < 0 || oy >= a.H || ox < 0 || ox >= a.W) continue;
              float x[CE];
              tr::unpack(*(const u32x4_t*)(s_cb + (cy * CW + cx) * CBP + cg * 16), x);
#pragma unroll
              for (int e = 0; e < CE; ++e) mx[e] = fmx_raw(mx[e], x[e]);
            }
        }
        *(u32x4_t*)((T*)a.fire_out[which] + (long long)n * a.fire_sN[which] + (long long)(gy * a.PW + gx) * a.fire_sP[which] + k0) = tr::pack(mx);
      }
      __syncthreads();                                             // the conv block is rewritten by the next tile
    };
    // block position of the first tap of this lane's pixel in chunk mc: the 1x1 expand reads the pixel itself, the 3x3 its window
    auto first_tap = [&](int which, int mc) __attribute__((always_inline)) -> const unsigned char* {
      const int m = mc * 64 + wave_m * 32 + l31;
      const int mm = m < npix ? m : 0;
      const int py = by_cw(mm), px = mm - py * CW;
      return s_sq + ((py + (which ? 0 : ring)) * PWd + px + (which ? 0 : ring)) * SQP + lhalf * 16;
    };
    if constexpr (KGS > 0) {
      // this share's tiles of one part, tiles_n apart; w holds the fragments of the first
      auto tiles = [&](int which, auto& w) __attribute__((always_inline)) {
        constexpr int TAPS = sizeof(w) / sizeof(u32x4_t) / KGS;
        if (j_first[which] * 64 >= a.fire_E[which]) return;
#pragma unroll 1
        for (int j = j_first[which];;) {
#pragma unroll 1
          for (int mc = 0; mc * 64 < npix; ++mc) {
            f32x4_t esc[4], esh[4];
            if constexpr (KGS < 4) load_affine(which, j, esc, esh);   // (before the MFMAs, which cover its latency, where the registers allow it)
            const unsigned char* pa = first_tap(which, mc);
            f32x16_t acc;
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[e] = 0.f;
            // pixel fragments one group of taps ahead; the barriers keep the scheduler from requesting all of them at once, which
            // takes the registers of the second workgroup
            constexpr int GT = TAPS == 9 && KGS <= 2 ? 3 : 1, NG = TAPS / GT;
            u32x4_t fa[2][GT * KGS];
            auto fetch = [&](int g) __attribute__((always_inline)) {
#pragma unroll
              for (int f = 0; f < GT * KGS; ++f) {
                const int tap = g * GT + f / KGS;
                fa[g & 1][f] = *(const u32x4_t*)(pa + ((tap / 3) * PWd + tap % 3) * SQP + (f % KGS) * 32);
              }
            };
            fetch(0);
#pragma unroll
            for (int g = 0; g < NG; ++g) {
              if (g + 1 < NG) fetch(g + 1);
#pragma unroll
              for (int f = 0; f < GT * KGS; ++f)
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, w[g * GT * KGS + f]), __builtin_bit_cast(bf16x8_t, fa[g & 1][f]), acc, 0, 0, 0);
              __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (KGS == 4) load_affine(which, j, esc, esh);
            tile_epilogue(which, j, mc, acc, esc, esh);
          }
          if constexpr (POOL) tile_pool(which, j);
          j += a.tiles_n;
          if (j * 64 >= a.fire_E[which]) break;
          load_w(which, j, w, f_begin, std::integral_constant<int, TAPS * KGS>());   // (here and not at the top, which would keep w over the pooling)
        }
      };
      u32x4_t w1[9 * KGS];
      load_w(1, gz, w1, f_begin, f_ahead9);
      tiles(0, w0);
      load_w(1, gz, w1, f_ahead9, f_end9);
      tiles(1, w1);
      __syncthreads();                                             // the squeeze block and the stages are rewritten
    } else {
#pragma unroll 1
    for (int which = 0; which < 2; ++which) {                      // 0: the 1x1 expand, 1: the 3x3 expand
      const int taps = which ? 9 : 1, E = a.fire_E[which];
      const int WP = fire_w_pitch(taps, S, ESZ), wrow_b = taps * S * ESZ;   // LDS pitch and bytes of a channel's weights
#pragma unroll 1
      for (int j = which ? j_first[1] : j_first[0]; j * 64 < E; j += a.tiles_n) {
        {   // the tile's weights: 64 channels x taps x S, contiguous in memory (rows beyond E are zero)
          const unsigned char* src = (const unsigned char*)a.fire_w[which] + (long long)j * 64 * wrow_b;
          const int cpr = wrow_b / 16, total = 64 * cpr;
          const SmallDiv by_cpr(cpr);
          // six requests per thread before the first is written to LDS: as a loop of load-then-store the copy paid one
          // memory latency per 4 KB (timestamps inside the kernel: 3.2 us for the 72 KB of a 3x3 tile over 64 channels)
          constexpr int CB = 6;
          for (int idx0 = tid; idx0 < total; idx0 += CB * NT) {
            u32x4_t wv[CB];
#pragma unroll
            for (int u = 0; u < CB; ++u) {
              const int idx = idx0 + u * NT;
              wv[u] = *(const u32x4_t*)(src + (long long)(idx < total ? idx : 0) * 16);   // (the tile is contiguous in memory)
            }
#pragma unroll
            for (int u = 0; u < CB; ++u) {
              const int idx = idx0 + u * NT, row = by_cpr(idx), c = idx - row * cpr;
              if (idx < total) *(u32x4_t*)(s_b + row * WP + c * 16) = wv[u];
            }
          }
        }
        __syncthreads();
#pragma unroll 1
        for (int mc = 0; mc * 64 < npix; ++mc) {
          f32x4_t esc[4], esh[4];
          load_affine(which, j, esc, esh);
          const unsigned char* pa = first_tap(which, mc);
          const unsigned char* pb = s_b + (wave_n * 32 + l31) * WP + lhalf * 16;
          f32x16_t acc;
#pragma unroll
          for (int e = 0; e < 16; ++e) acc[e] = 0.f;
#pragma unroll 1
          for (int tap = 0; tap < taps; ++tap) {
            const unsigned char* ta = pa + ((tap / 3) * PWd + tap % 3) * SQP;
            const unsigned char* tb = pb + tap * S * ESZ;
            for (int kg = 0; kg < kgs; ++kg) {
              const u32x4_t fa = *(const u32x4_t*)(ta + kg * 32), fb = *(const u32x4_t*)(tb + kg * 32);
#pragma unroll
              for (int e = 0; e < 4; ++e)
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(fb[e]), __uint_as_float(fa[e]), acc, 0, 0, 0);
            }
          }
          tile_epilogue(which, j, mc, acc, esc, esh);
        }
        if constexpr (POOL) tile_pool(which, j);
        else __syncthreads();                                      // the weight tile is rewritten
      }
    }
    }
  }
}

template <typename T, bool POOL, int TAPS1, int KGS>
static int launch_fire_kgs(const ConvArgs& a, int lds, hipStream_t st) {
  static std::atomic<bool> raised{false};
  const hipError_t e = raise_lds_limit(fire_kernel<T, POOL, TAPS1, KGS>, raised);
  if (e != hipSuccess) return (int)e;
  ConvArgs b = a;
  b.set_quotients();
  hipLaunchKernelGGL((fire_kernel<T, POOL, TAPS1, KGS>), dim3(a.grid < a.ntiles ? a.grid : a.ntiles), dim3(NT), lds, st, b);
  return (int)hipGetLastError();
}

template <typename T, bool POOL, int TAPS1>
static int launch_fire_inst(const ConvArgs& a, int lds, hipStream_t st) {
  if constexpr (sizeof(T) == 2) {
    switch (a.K / 16) {
      case 1: return launch_fire_kgs<T, POOL, TAPS1, 1>(a, lds, st);
      case 2: return launch_fire_kgs<T, POOL, TAPS1, 2>(a, lds, st);
      case 3: return launch_fire_kgs<T, POOL, TAPS1, 3>(a, lds, st);
      case 4: return launch_fire_kgs<T, POOL, TAPS1, 4>(a, lds, st);
    }
    return (int)hipErrorInvalidValue;
  } else {
    return launch_fire_kgs<T, POOL, TAPS1, 0>(a, lds, st);
  }
}

template <typename T>
static int launch_fire_t(const ConvArgs& a, hipStream_t st) {
  constexpr int ESZ = (int)sizeof(T), BKE = Tr<T>::BKE, CE = Tr<T>::CE;
  const bool pool = a.pool != POOL_NONE;
  // what the kernel assumes, checked again on the host
  // the first convolution: 1x1 / pad 0, or 3x3 / pad 1 with the taps of a channel chunk packed in consecutive steps
  const bool first3 = a.R == 3;
  if (a.mode != M_FLAT || a.has_res || a.ksplit >= 1 || a.ileave || a.pair || a.dw_panel || a.pwdw || a.dw_w || a.stride != 1 || a.R != a.S ||
      (first3 ? (a.pad != 1 || !a.kchunk || a.C % BKE != 0 || a.Kred_pad != 9 * a.C || a.H > 0xffff || a.W > 0xffff)
              : (a.R != 1 || a.pad != 0 || a.kchunk || a.Kred_pad < (a.C + BKE - 1) / BKE * BKE)) ||
      a.C % CE != 0 || a.C < CE || a.Kred_pad % BKE != 0 ||
      a.K < 1 || a.K > 64 || (a.K * ESZ) % 32 != 0 || a.OH != a.H || a.OW != a.W ||
      (a.fire_E[0] < 1 && a.fire_E[1] < 1) ||
      a.tiles_n < 1 || a.fire_skip != (a.fire_E[1] + 63) / 64 % a.tiles_n || a.tiles_m != a.N * a.tiles_y * a.tiles_x || a.ntiles != a.tiles_m * a.tiles_n || a.grid < 1 ||
      a.in_sN < 0 || a.in_sH < 0 || a.in_sW < a.C)
    return (int)hipErrorInvalidValue;
  for (int e = 0; e < 2; ++e) {   // a part with no channels does not exist (a ConvX -> ConvY pair instead of a module)
    if (a.fire_E[e] == 0) continue;
    if (!a.fire_w[e] || !a.fire_scale[e] || !a.fire_shift[e] || !a.fire_out[e] || a.fire_E[e] < CE || a.fire_E[e] % CE != 0 ||
        a.fire_sP[e] < a.fire_E[e] || a.fire_sP[e] % CE != 0 || a.fire_sN[e] % CE != 0 || ((uintptr_t)a.fire_out[e] & 15) || ((uintptr_t)a.fire_w[e] & 15))
      return (int)hipErrorInvalidValue;
  }
  int ch, cw, pool_pos = 0;
  if (pool) {
    // max-pooling with windows of 2 or 3 at stride 2, no padding; every window starts inside the map
    if (a.pool != POOL_MAX || a.pk < 2 || a.pk > 3 || a.ps != 2 || a.pp != 0 || a.pph < 1 || a.ppw < 1 || a.PH < 1 || a.PW < 1 ||
        (a.PH - 1) * a.ps >= a.H || (a.PW - 1) * a.ps >= a.W ||
        a.tiles_y != (a.PH + a.pph - 1) / a.pph || a.tiles_x != (a.PW + a.ppw - 1) / a.ppw)
      return (int)hipErrorInvalidValue;
    ch = (a.pph - 1) * a.ps + a.pk; cw = (a.ppw - 1) * a.ps + a.pk;
    pool_pos = ch * cw;
  } else {
    if (a.th < 1 || a.tw < 1 || a.tiles_y != (a.H + a.th - 1) / a.th || a.tiles_x != (a.W + a.tw - 1) / a.tw) return (int)hipErrorInvalidValue;
    ch = a.th; cw = a.tw;
  }
  const int ring = a.fire_E[1] > 0 ? 1 : 0;
  const int positions = (ch + 2 * ring) * (cw + 2 * ring);
  const int lds = fire_lds(positions, a.K, ESZ, pool_pos);
  if (positions > kFireMaxPositions || lds > 160 * 1024 || !block_window_fits(a, ch + 2 * ring + a.R - 1, ESZ)) return (int)hipErrorInvalidValue;
  if (first3) return pool ? launch_fire_inst<T, true, 9>(a, lds, st) : launch_fire_inst<T, false, 9>(a, lds, st);
  return pool ? launch_fire_inst<T, true, 1>(a, lds, st) : launch_fire_inst<T, false, 1>(a, lds, st);
}

int launch_fire(const ConvArgs& a, int dtype, void* stream) {
  return dtype == DT_BF16 ? launch_fire_t<bf16_t>(a, (hipStream_t)stream) : launch_fire_t<float>(a, (hipStream_t)stream);
}

size_t fire_lds_bytes(int conv_h, int conv_w, int S, int esz, int pooled, int ring) {
  return (size_t)fire_lds((conv_h + 2 * ring) * (conv_w + 2 * ring), S, esz, pooled ? conv_h * conv_w : 0);
}

}  // namespace xenos
