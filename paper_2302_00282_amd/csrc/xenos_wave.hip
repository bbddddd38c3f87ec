// gfx950 (CDNA4) kernel of small dense convolution chains:
//
//  conv_wave_kernel   implicit-GEMM convolution chain (any kernel size and stride) in tiles of 32 pixels x 32 channels, the reduction of a tile shared out over the four wavefronts of its workgroup
//                     (wave_gemm.h); scale / shift, shortcut and ReLU in the sum of the partial tiles, or raw sums for a reduction
//                     that is split over workgroups too.
#include "wave_gemm.h"

namespace xenos {

// What the kernel needs, in the order and form it needs it: four lines of the constant cache, read at once, where the general
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
template <typename T, bool UNI, bool DIRECT>
__global__ __launch_bounds__(NT, 4) void conv_wave_kernel(const WaveConvArgs a) {
  FETCH_ARGS(WaveConvArgs);
  using tr = Tr<T>;
  using tile = WaveTile<T, 1>;
  constexpr int CE = tr::CE, BKE = tr::BKE, ESZ = (int)sizeof(T);
  extern __shared__ __align__(16) unsigned char smem[];
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
      const int m = (int)tm * 32 + (lane & 31);
      const int img = small_quotient(m, a.r_ohw), p = m - img * a.OHW, oh = small_quotient(p, a.r_ow), ow = p - oh * a.OW;
      const int ih = m < a.M ? oh * a.stride - a.pad : -0x4000, iw = ow * a.stride - a.pad;
      off = (int)((unsigned)img * a.sN + (unsigned)ih * a.sH + (unsigned)iw * a.sW);
      yx = (int)(((unsigned)ih << 16) | ((unsigned)iw & 0xffffu));
    }
    int aoff[4], ayx[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      aoff[j] = __builtin_amdgcn_ds_bpermute((j * 8 + lrow) * 4, off) + (UNI ? ch[j & 1] * 16 : 0);
      ayx[j] = __builtin_amdgcn_ds_bpermute((j * 8 + lrow) * 4, yx);
    }
    const unsigned woff[2] = {lrow * a.wpitch + ch[0] * 16u, lrow * a.wpitch + ch[1] * 16u};
    const rsrc_t wb = make_window((const unsigned char*)a.w + (size_t)tn * 32 * a.wpitch, kWindow);
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
      for (int j = 0; j < 4; ++j) {
        const int y = (ayx[j] >> 16) + kr[j & 1], x = (int)(short)ayx[j] + kc[j & 1];
        const bool ok = ((unsigned)y < (unsigned)a.H) & ((unsigned)x < (unsigned)a.W) & kok[j & 1];
        unsigned o = ok ? (unsigned)aoff[j] + koff[j & 1] : kNoLoad;
        asm volatile("" : "+v"(o));
        if constexpr (DIRECT) load_to_lds(wa, dst + j * 1024, o, 0);
        else *(u32x4_t*)(dst + j * 1024 + lane * 16) = load_window(wa, o);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) load_to_lds(wb, dst + 4096 + j * 1024, woff[j & 1], j * 8 * a.wpitch + s * ROWB);
    };
    tile::begin(n, a.stages, s_w, request);

    // what the epilogue reads: on its way during the reduction.  The thread finishes channels k .. k + 3 of pixel row m
    const int row = tid >> 3, c = (tid & 7) * 4, m = (int)tm * 32 + row, k = (int)tn * 32 + c;
    const bool live = m < a.M && k < a.K;
    const int img = small_quotient(m, a.r_ohw), p = m - img * a.OHW;
    f32x4_t sc = {}, sh = {};
    u32x4_t res = {};                                              // (as they lie in memory: converted behind the reduction)
    if (!(a.flags & WF_PARTIAL)) {
      sc = *(const f32x4_t*)(a.scale + k);
      sh = *(const f32x4_t*)(a.shift + k);
    }
    if (a.res) {                                                   // (uniform)
      unsigned o = live ? (unsigned)img * a.res_sN + (unsigned)p * a.res_sP + k * ESZ : kNoLoad;
      asm volatile("" : "+v"(o));
      const rsrc_t wr = make_window(a.res, kWindow);
      if constexpr (ESZ == 2) {
        const uint2 r = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(wr, (int)o, 0, 0));
        res[0] = r.x; res[1] = r.y;
      } else {
        res = load_window(wr, o);
      }
    }
    f32x16_t acc[1];
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[0][e] = 0.f;
    tile::finish(n, a.stages, s_w, request, acc);
    __syncthreads();
    f32x4_t v = tile::sum(smem, wave_bytes, row, c);
    if (live) {
      if (a.flags & WF_PARTIAL) {
        *(f32x4_t*)((float*)a.out + ((size_t)z * a.M + m) * a.part_ld + k) = v;
      } else {
        v = v * sc + sh;
        if (a.res) {
          if constexpr (ESZ == 2) v += f32x4_t{bf2f((uint16_t)res[0]), __uint_as_float(res[0] & 0xffff0000u), bf2f((uint16_t)res[1]), __uint_as_float(res[1] & 0xffff0000u)};
          else v += __builtin_bit_cast(f32x4_t, res);
        }
        if (a.flags & WF_RELU) {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = fmx(v[e], 0.f);
        }
        unsigned char* dst = (unsigned char*)a.out + (size_t)((unsigned)img * a.out_sN + (unsigned)p * a.out_sP);
        if (ESZ == 4 || (a.flags & WF_OUT_F32)) *(f32x4_t*)(dst + k * 4) = v;
        else *(uint2*)(dst + k * 2) = uint2{f2bf2(v[0], v[1]), f2bf2(v[2], v[3])};
      }
    }
    __syncthreads();                                               // the partial tiles are rewritten
  }
}

size_t conv_wave_lds(int stages) { return (size_t)4 * stages * WaveTile<float, 1>::STAGE; }

// Steps of a wavefront that are on their way at a time: up to four where a unit has one workgroup, two where it has two, one where it has
// more, which then hide each other's latency (3x3 layers in bf16, four in a row: 128 channels 28x28 batch 4, 392 tiles, four 36.8 us, two
// 25.9; 256 channels 14x14 batch 16, 784 tiles, two 60.8, one 56.2; 400 tiles of 144 steps, two 51.8, one 58.5)
int conv_wave_stages(int steps, int tiles) {
  const int n = (steps + 3) / 4, most = tiles <= 256 ? 4 : tiles <= 512 ? 2 : 1;
  return n < 1 ? 1 : n < most ? n : most;
}

template <typename T, bool UNI, bool DIRECT>
static int launch_conv_wave_inst(const WaveConvArgs& w, int grid, int lds, hipStream_t st) {
  static std::atomic<bool> raised{false};
  const hipError_t e = raise_lds_limit(conv_wave_kernel<T, UNI, DIRECT>, raised);
  if (e != hipSuccess) return (int)e;
  hipLaunchKernelGGL((conv_wave_kernel<T, UNI, DIRECT>), dim3(std::min((uint32_t)grid, w.tiles)), dim3(NT), lds, st, w);
  return (int)hipGetLastError();
}

template <typename T>
static int launch_conv_wave_t(const ConvArgs& a, hipStream_t st) {
  constexpr int ESZ = (int)sizeof(T), BKE = Tr<T>::BKE;
  const bool partial = a.ksplit >= 1;
  const int ks = partial ? a.ksplit : 1;
  // what the kernel assumes, checked again on the host
  if (!conv_wave_takes(a, ESZ) || a.dw_w || a.pair || a.ileave || a.pool != POOL_NONE || a.tiles_m != (a.M_total + 31) / 32 || a.tiles_n != (a.K + 31) / 32 ||
      (!partial && (a.out_sK != 1 || (a.has_res && (!a.vec_res || !a.res)))) ||
      (partial && (!a.part || a.part_ld < a.tiles_n * 32 || a.steps_per_split < 1)) || a.grid < 1)
    return (int)hipErrorInvalidValue;
  WaveConvArgs w{};
  w.in = a.in; w.w = a.w; w.scale = a.scale; w.shift = a.shift; w.res = !partial && a.has_res ? a.res : nullptr; w.out = partial ? (void*)a.part : a.out;
  w.nz = (uint32_t)(a.tiles_n * ks); w.m_nz = host_multiplier(w.nz); w.ks = (uint32_t)ks; w.m_ks = host_multiplier(w.ks);
  w.tiles = (uint32_t)a.tiles_m * w.nz;
  w.nsteps = a.Kred_pad / BKE; w.steps_per_share = partial ? a.steps_per_split : w.nsteps;
  w.rs = (uint32_t)(a.R * a.S); w.m_rs = host_multiplier(w.rs); w.S = (uint32_t)a.S; w.m_S = host_multiplier(w.S); w.r_C = 1.f / (float)a.C; w.r_S = 1.f / (float)a.S;
  w.M = a.M_total; w.OHW = a.OH * a.OW; w.OW = a.OW; w.r_ohw = 1.f / (float)w.OHW; w.r_ow = 1.f / (float)w.OW;
  w.stride = a.stride; w.pad = a.pad; w.H = a.H; w.W = a.W; w.C = a.C;
  w.sN = (uint32_t)(a.in_sN * ESZ); w.sH = (uint32_t)(a.in_sH * ESZ); w.sW = (uint32_t)(a.in_sW * ESZ); w.wpitch = (uint32_t)(a.Kred_pad * ESZ);
  w.K = a.K; w.part_ld = a.part_ld; w.flags = (a.relu ? WF_RELU : 0) | (partial ? WF_PARTIAL : 0) | (a.out_f32 ? WF_OUT_F32 : 0);
    const int osz = a.out_f32 ? 4 : ESZ;
  w.out_sN = (uint32_t)(a.out_sN * osz); w.out_sP = (uint32_t)(a.out_sP * osz); w.res_sN = (uint32_t)(a.res_sN * ESZ); w.res_sP = (uint32_t)(a.res_sP * ESZ);
  w.stages = conv_wave_stages(w.steps_per_share, (int)w.tiles);
  const int lds = (int)conv_wave_lds(w.stages);
  const bool direct = ((uintptr_t)a.in & 15) == 0;
  if (a.R * a.S == 1 || a.kchunk)
    return direct ? launch_conv_wave_inst<T, true, true>(w, a.grid, lds, st) : launch_conv_wave_inst<T, true, false>(w, a.grid, lds, st);
  return direct ? launch_conv_wave_inst<T, false, true>(w, a.grid, lds, st) : launch_conv_wave_inst<T, false, false>(w, a.grid, lds, st);
}

int launch_conv_wave(const ConvArgs& a, int dtype, void* stream) {
  return dtype == DT_BF16 ? launch_conv_wave_t<bf16_t>(a, (hipStream_t)stream) : launch_conv_wave_t<float>(a, (hipStream_t)stream);
}

}  // namespace xenos
