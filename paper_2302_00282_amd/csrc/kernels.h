// Launch descriptors shared by the host planner/runtime and the gfx950 kernels.
// Everything here is plain data: the planner fills these at plan time, the runtime patches
// the external input/output pointers and launches.
#pragma once
#include <stddef.h>
#include <stdint.h>
#include <algorithm>
#include <cmath>
#include "index_div.h"

namespace xenos {

enum { DT_F32 = 0, DT_BF16 = 1 };

// Bytes of one tile row consumed per reduction step of the dense-conv kernel (64 bf16 / 32 fp32 elements).
// The packed weight layout depends on it, so host and kernels share the constant.
constexpr int kRowBytes = 128;

// How the rows (m) of an implicit-GEMM tile enumerate conv-output pixels.  The enumeration IS the
// linked dataflow of Section 4.1 / Figure 4: the producer walks pixels in the order its linked
// consumer (the pooling) reads them.
enum {
  M_FLAT = 0,     // m = (n*OH + oh)*OW + ow: no pooling, output written pixel-major
  M_ZIGZAG = 1,   // m = 4*window + (dy*2+dx): 2x2/s2 pooling windows are 4 consecutive rows (Figure 4 zig-zag)
  M_PATCH = 2,    // tile = spatial patch of one image, staged on chip, then pooled (any k/s/pad/ceil)
  M_GAP = 3       // tile = (image, channel tile); loops over the whole map, global average in registers
};

enum { POOL_NONE = 0, POOL_MAX = 1, POOL_AVG = 2, POOL_GAP = 3 };

// Tile configurations of the dense-conv kernel (block = 256 threads = 4 wavefronts).
struct TileCfg { int bm, bn, wm, wn; };
static const TileCfg kTileCfgs[] = {
  {128, 128, 64, 64},
  {128, 64, 64, 32},
  {64, 64, 32, 32},
  {32, 128, 32, 32},
};
static const int kNumTileCfgs = 4;
// Configuration index of the halo-staged 3x3 kernel: 256 pixels x 128 or 64 channels, 512 threads, TH x TW spatial tile.
static const int kHaloCfg = 4;
// Configuration index of the first-layer kernel: 32 pixels x K (32 or 64) channels per wavefront, the reduction
// C*R*S (at most kStemRed, in up to kStemPasses MFMA passes of 32) gathered straight from the graph input through `ktab`.
static const int kStemCfg = 5;
static const int kStemPasses = 5;
static const int kStemRed = 32 * kStemPasses;
// Configuration index of the kernel that links the first two 3x3 convolutions (intermediate tensor kept in LDS): at most
// 4 input channels -> kPairChannels -> kPairChannels; the first convolution reduces over kPairRed slots = tap * 4 + channel.
static const int kPairCfg = 6;
// Configuration index of the kernel that streams the weights of a fully connected chain with at most 32 rows (128 channels per
// workgroup, reduction shared out over workgroups; always followed by the summing pass)
static const int kFcCfg = 7;
static const int kFcChannels = 128;
// Configuration index of the first-layer kernel that stages its input block in LDS (bf16 path, or fp32 with a pooling; fp32 NCHW graph input with at most 4
// channels, square kernel up to 7x7, stride 1 or 2): tiles of kStemLdsTh x kStemLdsTw output pixels of one image
static const int kStemLdsCfg = 8;
static const int kStemLdsPph = 3, kStemLdsPpw = 8;   // pooling windows per tile when a max-pooling is linked
static const int kStemLdsTh = 8, kStemLdsTw = 16, kStemLdsInMax = 784;   // (7 * 2 + 7) x (15 * 2 + 7) = 777 positions at most
// (per kernel size class the kernel is instantiated for, by taps: up to 3x3 at stride 2 a block is at most 17 x 33 or 15 x 35
// positions, up to 5x5 19 x 35)
constexpr int stem_lds_in_positions(int taps) { return taps <= 12 ? 576 : taps <= 28 ? 672 : kStemLdsInMax; }
constexpr int stem_lds_steps(int taps) { return taps <= 12 ? 3 : taps <= 28 ? 7 : 13; }          // steps of four taps
constexpr int stem_lds_rounds(int taps) { return (stem_lds_in_positions(taps) + 255) / 256; }    // positions of the block per thread of 256
// LDS of the kernel for 32 or 64 output channels: two input blocks of four-channel positions, the staging slices of four wavefronts (32
// pixels, pitch an odd number of 16-byte slots), scale and shift, the tap offsets of either lane half.  The kernel asserts the same
constexpr size_t stem_lds_bytes(int taps, int channels, int esz) {
  return (size_t)2 * stem_lds_rounds(taps) * 256 * 4 * esz + 4 * 32 * (channels * esz + 16) + 2 * channels * 4 + stem_lds_steps(taps) * 2 * 8;
}
// Workgroups of the kernel that a compute unit holds, by its registers and LDS (a test compares them with the code objects'): as many are
// launched, so that none starts, with its weights and tables, behind another, and none is missing to hide the others' latencies.
// Batch 8 to 32, one fewer and one more than this: 32 channels 3x3 bf16 1.05 times the time, fp32 1.05 / 1.12; 5x5 bf16 1.07 / 1.13,
// fp32 1.06 / 1.12; 64 channels 3x3 bf16 1.02, 5x5 1.02 / 1.08, 7x7 1.22 with one more.
// 3x3 bf16 without a pooling, 24 and 32 channels, batch 8 to 64: five instead of four 0.97 to 1.015, 0.99 on average.
constexpr int stem_lds_resident(int taps, int channels, int esz, bool pool) {
  if (esz == 4) return channels > 32 ? 2 : 3;
  return taps <= 12 ? (channels > 32 || pool ? 4 : 5) : taps <= 28 ? (channels > 32 || pool ? 3 : 4) : channels > 32 || pool ? 2 : 3;
}
// Configuration index of the kernel that links a pointwise (1x1) convolution chain with the depthwise 3x3 chain that consumes
// it: a TH x TW block of depthwise output pixels x kPwDwChannels channels per workgroup, the pointwise output of the block
// (+ halo) staged in LDS, at most kPwDwMaxPositions positions
static const int kPwDwCfg = 9;
static const int kPwDwChannels = 64, kPwDwMaxPositions = 400;
// Configuration index of the kernel that runs a Fire module (squeeze 1x1 -> expand 1x1 || expand 3x3 -> concat [-> max-pooling])
// as one chain: the squeeze output of a tile (+ halo, at most kFireMaxPositions positions, at most 64 channels) stays in LDS
static const int kFireCfg = 10;
static const int kFireMaxPositions = 400;
// Configuration index of the kernel that runs pointwise -> depthwise 3x3 -> pointwise as one chain, a tile of output pixels x all
// channels per workgroup
static const int kUnitCfg = 11;
// Configuration index of the kernel for chains of few pixels (fp32 at link level 3: of any number): tiles of kWaveRows pixels x kWaveChannels channels, the reduction of a tile
// shared out over the wavefronts of its workgroup
static const int kWaveCfg = 12;
static const int kWaveRows = 32, kWaveChannels = 32;
constexpr int kWaveStageF32 = 32 * 128 + 3 * 32 * 64;   // fp32: LDS of a step, 32 pixel rows and the three bf16 parts of 32 channel rows
// fp32 operands of the wave kernels are taken apart as multiples of 2^-24: the smallest number of fp32, 2^-149, then is a normal number of bf16 (2^-126 and
// more), so that three parts hold every number below 2^103, and its products what fp32 would hold of them and more
constexpr float kWavePartScale = 16777216.f;
constexpr unsigned kWavePartMostBits = (127u + 103u) << 23;      // 2^103
constexpr unsigned short kWaveWholeWeight = 0x7fc0;   // in the place of a weight's upper part: the other two are the halves of the fp32 number itself
static const int kWave64Cfg = 13;      // the same in tiles of 64 x 64
// Configuration index of the kernel that computes a first layer's 2x2 pooling windows on the vector unit, a window x kFirstChannels channels per thread
static const int kFirstCfg = 15;
constexpr int kFirstChannels = 8;
// Configuration index of the 3x3 kernel whose weights go from the cache into registers (bf16)
static const int kFrag3Cfg = 14;
constexpr int kFrag3Pitch = 80;        // LDS bytes of a patch position: 32 channels and an odd number of 16-byte slots
// positions of the patch in LDS, for blocks per wavefront x pixel groups; row pitch of the patch
constexpr int frag3_positions(int pb, int wp) { return wp == 2 ? 384 : pb > 7 ? 320 : pb > 4 ? 192 : 128; }
constexpr int frag3_pitch(int tw) { return (tw + 2 + 1) / 4 * 4 + 2; }
constexpr size_t frag3_lds(int pb, int wp, int ks) {
  return (size_t)ks * 2 * frag3_positions(pb, wp) * kFrag3Pitch + wp * pb * 16 * 4 + (ks > 1 ? 4 / (wp * ks) * pb * 2048 : 0);
}
static const int kFcWgPerCu = 1;
static const int kFcDirectSteps = 16;   // reductions of at most this many 64-element steps are not shared out (no summing pass)    // workgroups per compute unit the reduction split of such a chain aims at
static const int kPairChannels = 64, kPairRed = 48;
static const int kPairRows = 128, kPairPatchMax = 180;   // output pixels and patch positions ((TH+2) x 18) of a tile
static const int kPairInMax = 256;   // positions of the staged block of the graph input, (TH+4) x (TW+4) plus slack for the pitch columns
static const int kHaloRows = 256, kHaloCols = 128, kHaloPatchMax = 360;
static const long long kL2BytesPerXcd = 4ll << 20;   // gfx950: one 4 MB L2 per XCD
// the staged patch has one of two fixed row pitches (pixels): tiles up to 16 or up to 32 pixels wide
static const int kHaloPitchTiny = 10, kHaloPitchNarrow = 18, kHaloPitchWide = 34;

struct ConvArgs {
  const void* in;        // activations: NHWC in the compute type (vector loader), or any strided fp32/T tensor (scalar loader)
  const void* w;         // packed weights [Kout_pad][Kred_pad] in the compute type, reduction index = (r*S+s)*C + c
  const float* scale;    // folded per-channel scale [Kout_pad] (1 where no BN)
  const float* shift;    // folded per-channel shift [Kout_pad]
  const void* res;       // residual (NHWC view, compute type) or nullptr
  const void* zeros;     // 256 bytes of zeros in device memory: what a masked 16-byte load reads (dwpw_kernel)
  void* out;
  const int32_t* ktab;   // scalar loader only: per reduction index {offset, (r<<16)|s}
  int N, C, H, W;
  long long in_sN, in_sH, in_sW;   // element strides of the input view (channel stride is 1 for the vector loader)
  int in_f32;            // scalar loader: input elements are fp32 (graph input) instead of the compute type
  int K, R, S, stride, pad, OH, OW;
  int Kred, Kred_pad;    // R*S*C and its padding to the reduction step
  int wfrag;             // weights in fragment order: [32-channel block][step][k-group][lane][16 bytes]
  int kchunk;            // reduction order: 1 = (channel chunk, r, s, channel in chunk), needs C % step == 0; 0 = (r, s, c)
  int mode;              // M_*
  int relu, has_res;
  // != 0: the chain also performs the two-group channel shuffle of the concat it ends in.  `res` is the other part of the
  // concat (strides res_sN / res_sP), `out` the concat buffer (2 K channels per pixel); channel k of this chain is stored
  // at output channel 2k + (ileave - 1) and channel k of the other part at 2k + (2 - ileave).  M_FLAT, general and
  // depthwise-panel kernels, 16-byte aligned channel groups only.
  int ileave;
  long long res_sN, res_sP;        // residual strides (image, pixel); channel stride 1
  int pool, pk, ps, pp, PH, PW, cip;   // linked pooling (POOL_*), window, stride, pad, pooled size, count_include_pad
  int patch_h, patch_w, pph, ppw, patches_y, patches_x;   // M_PATCH geometry (conv-output patch, pooled patch)
  long long out_sN, out_sP, out_sK;    // output strides (image, pixel, channel) in elements
  int out_f32;           // store fp32 instead of the compute type (graph output)
  int vec_out, vec_res;  // 16-byte channel-group stores / shortcut loads are legal (alignment, unit channel stride, K % group == 0)
  // linked depthwise producer (nullptr = none): `in` is then the depthwise INPUT (NHWC), H x W the depthwise output
  const void* dw_w; const float* dw_scale; const float* dw_shift;   // [k*k][C] compute type, folded scale / shift [C]
  int dw_k, dw_stride, dw_pad, dw_H, dw_W, dw_relu;
  long long dw_sN, dw_sP;
  // linked first-layer producer (pair kernel): `in` is the caller's fp32 NCHW tensor (unit stride along W) with pair_C
  // channels, dw_w its packed weights [kPairChannels][kPairRed], dw_scale / dw_shift / dw_relu its epilogue; C, H, W
  // describe the intermediate tensor
  int pair, pair_C;
  long long pair_sN, pair_sC, pair_sH;
  int dw_panel;          // > 0: the depthwise result of a whole panel of this many channels is staged in LDS (dwpw_kernel)
  // linked depthwise CONSUMER (pwdw_kernel): this 1x1 / stride 1 chain's output tile stays in LDS and a depthwise 3x3 chain
  // (dw_w [9][K], dw_scale / dw_shift [K], dw_stride, dw_pad = 1, dw_relu) runs out of it; H x W is the pointwise map,
  // OH x OW the depthwise output, th x tw the tile of depthwise output pixels, tiles_y x tiles_x the tile grid per image.
  // 2: maps of few pixels, on pwdw_wave_kernel (a workgroup takes 32 of a tile's 64 channels)
  int pwdw;
  // linked Fire module (fire_kernel): this 1x1 / stride 1 chain is the squeeze (K <= 64 channels); its output tile (+ halo)
  // stays in LDS and two expand chains read it there: [0] 1x1, [1] 3x3 / pad 1.  fire_w: [E padded to 64][taps][K] in the
  // compute type; fire_scale / fire_shift: folded epilogue, padded to 64; fire_out: where each part goes (NHWC view of the
  // compute type: image stride fire_sN, pixel pitch fire_sP), after the linked max-pooling (pool, pk, ps, pp, PH, PW; tiles of
  // pph x ppw windows) if there is one; th x tw = tile of output pixels otherwise; tiles_n = channel shares
  int fire;
  const void* fire_w[2]; const float* fire_scale[2]; const float* fire_shift[2];
  void* fire_out[2]; long long fire_sN[2], fire_sP[2];
  int fire_E[2], fire_relu[2];
  int fire_skip;         // 64-channel tiles of the 3x3 part modulo the shares: share fire_skip takes the 1x1 part's first
  // linked unit (unit_kernel): this chain is the second pointwise convolution of pointwise -> depthwise 3x3 -> pointwise; `in` is
  // the input of the first (unit_C channels, weights fire_w[0] in fragment order with a reduction padded to unit_kred, epilogue
  // fire_scale / fire_shift / fire_relu[0]), C the channels of the depthwise convolution (dw_*) over the dw_H x dw_W map,
  // th x tw the tile of output pixels
  int unit, unit_C, unit_kred;
  // reduction split across workgroups (ksplit >= 1, M_FLAT only; 0 = none): share z covers steps [z*steps_per_split, ...)
  // and writes raw fp32 sums to part[z][m][k] (row pitch part_ld); a splitk_finish pass completes the chain
  int ksplit, steps_per_split, part_ld;
  float* part;
  int th, tw, tiles_y, tiles_x;   // halo kernel: spatial tile and tile grid over the stacked padded rows n*(H+2)+oh
  int halo_bn;           // halo kernel: output channels per tile (128 or 64)
  int halo_mgroup;       // halo kernel: an XCD walks its pixel tiles in groups of this many, every output-channel tile of a group
                         // before the next group (>= 1; a value of at least the XCD's tile count = one sweep per channel tile)
  int frag3, frag3_wp, frag3_ks;   // conv3x3_frag_kernel: blocks of 16 pixels per wavefront, groups of pixels and shares of the reduction among its wavefronts
  int halo_plin;         // halo kernel: patch-linear rows (GEMM row = patch position, pitch TW + 2; pixel-major chains only)
  int M_total;           // rows enumerated over the whole problem (FLAT, ZIGZAG); per-image rows for GAP
  int tiles_m, tiles_n, ntiles;
  int xcd_m;             // dense-conv kernel: the 8 XCDs form an xcd_m x (8/xcd_m) grid over pixel tiles x (channel tiles x shares)
  int grid;              // workgroups launched (>= 1); tiles are visited with a stride of `grid`
  // multipliers of quotients (host_multiplier, 0: none) by tiles_m, tiles_y * tiles_x and tiles_x, set by the launchers of the kernels that use them.
  // (With both sides below 2^15 only, and the compiler's division beyond, 50000 tiles of pwdw_kernel took 2 to 5 % longer, of fire_kernel 3 %)
  uint32_t q_tm, q_sp, q_tx;
  uint32_t q_c, q_k;     // by the 32-channel blocks of C and K (unit_kernel: parts of at most 16 times as many)
  void set_quotients() {
    const long long cb = (C + 31) / 32, kb = (K + 31) / 32, sp = (long long)tiles_y * tiles_x;
    q_tm = host_multiplier(ntiles, tiles_m); q_sp = host_multiplier(tiles_m, sp); q_tx = host_multiplier(sp, tiles_x);
    q_c = host_multiplier(16 * cb + 1, cb); q_k = host_multiplier(16 * kb + 1, kb);
  }
};

struct DwArgs {
  const void* in; const void* w;     // w: [R*S][C] in the compute type
  const float* scale; const float* shift;
  void* out;
  int N, C, H, W, R, S, stride, pad, OH, OW;
  long long in_sN, in_sP;            // NHWC view strides (image, pixel)
  long long out_sN, out_sP;
  int relu;
  long long total_vec;               // N*OH*OW*(C/vec)
};

// Stand-alone passes of the un-linked baselines (and of whatever the link pass could not absorb).
enum { ELT_AFFINE = 0, ELT_RELU = 1, ELT_ADD = 2, ELT_COPY = 3 };
struct EltArgs {
  const void* a; const void* b; void* out;
  const float* scale; const float* shift;
  int op, relu;                      // relu applied after op when set
  int C;                             // channels of the view
  long long pixels;                  // N*H*W
  long long a_sP, b_sP, out_sP;      // pixel strides of the NHWC views
  long long a_sK, out_sK;            // channel strides of a and out (1 except for the strided copies of a channel shuffle)
};

struct PoolArgs {
  const void* in; void* out;
  int N, C, H, W, OH, OW, k, s, p, kind, cip;   // kind: POOL_MAX / POOL_AVG / POOL_GAP
  long long in_sN, in_sP, out_sN, out_sP;
};

// Layout / type conversion at the graph boundary (the transpose operator of Table 3).
struct CvtArgs {
  const void* in; void* out;
  int N, C, H, W;
  int Cout;                          // channels written per pixel (>= C; channels C..Cout-1 are zero-filled)
  long long in_sN, in_sC, in_sP;     // element strides: image, channel, pixel (pixel index = h*W + w)
  long long out_sN, out_sC, out_sP;
  int in_f32, out_f32;
};

struct SplitKArgs {
  const float* part; int ksplit, part_ld;
  int M, K, OHW;                     // rows (n*OH*OW), output channels, pixels per image
  const float* scale; const float* shift;
  const void* res; long long res_sN, res_sP;
  void* out; long long out_sN, out_sP, out_sK;
  int relu, out_f32;
  int gap;                           // 1: average the finished pixels of every image (linked global average), out = [image][K]
};

// Launchers (defined in xenos_kernels.hip).  dtype = DT_*.  Return a hipError_t value as int.
int launch_conv(const ConvArgs& a, int dtype, int cfg, int scalar_loader, void* stream);
int launch_dw(const DwArgs& a, int dtype, void* stream);
int launch_elt(const EltArgs& a, int dtype, void* stream);
int launch_pool(const PoolArgs& a, int dtype, void* stream);
int launch_cvt(const CvtArgs& a, int dtype, void* stream);
int launch_splitk_finish(const SplitKArgs& a, int dtype, void* stream);
size_t conv_lds_bytes(int cfg, int mode);

// Bytes from the first input row that a tile of conv_kernel's (at most 128 of the chain's pixels, row by row, or a patch) touches to the
// end of what it reads, at most.  With pixels of two images the tile ends `rows` output rows into the second at most and began as many
// before the end of the first.
inline double conv_tile_span(const ConvArgs& a, int esz) {
  const bool flat = a.mode == M_FLAT, zig = a.mode == M_ZIGZAG;
  const double per = zig ? 4.0 * a.PH * a.PW : (double)a.OH * a.OW, line = zig ? 2.0 * a.PW : (double)a.OW;
  const double images = flat || zig ? std::min<double>(a.N, std::floor(127 / per) + 2) : 1;
  const double rows = a.mode == M_PATCH ? 128 : zig ? 2 * (std::floor(64 / line) + 2) : std::floor(127 / line) + 2;
  const double sN = (double)a.in_sN, sH = (double)a.in_sH;
  double span = (images - 1) * sN + a.H * sH;
  if (images == 1) span = std::min(span, (rows * a.stride + a.R) * sH);
  if (images == 2) span = std::min(span, std::max(0.0, sN - std::min((zig ? 2 * a.PH : a.OH) * a.stride, a.H) * sH) + (2 * rows * a.stride + a.R + a.pad) * sH);
  return (span + (double)a.W * (double)a.in_sW + a.C) * esz;
}
// Can the loader for reductions whose tap is uniform address them, and a tile's weight rows, with 32-bit offsets?
inline bool conv_window_fits(const ConvArgs& a, int esz) {
  const double lim = 0xffffff00ll;
  return a.in_sN >= 0 && a.in_sH >= 0 && a.in_sW >= 0 && conv_tile_span(a, esz) < lim && 128.0 * a.Kred_pad * esz < lim;
}
// Do `rows` rows of an image, from where a block of positions begins, and 64 rows of weights fit the windows of pw_gemm_phase?
constexpr unsigned kBlockWindow = 1u << 31;
inline bool block_window_fits(const ConvArgs& a, int rows, int esz) {
  return (double)a.in_sH * std::min(rows, a.H) * esz < kBlockWindow && 64.0 * a.Kred_pad * esz < 0xffffff00ll;
}
// Do a chain's sizes fit the indices of the wave kernel (quotients, packed coordinates and byte offsets of 32 bits)?
inline bool conv_wave_takes(const ConvArgs& a, int esz, int edge = kWaveRows) {
  const int bke = kRowBytes / esz, ce = 16 / esz;
  const double lim = 2147483648.0, tiles = std::ceil(a.M_total / (double)edge) * std::ceil(a.K / (double)edge) * (a.ksplit > 1 ? a.ksplit : 1);
  return a.mode == M_FLAT && a.C % ce == 0 && a.K % 4 == 0 && a.Kred_pad % bke == 0 && a.Kred_pad / bke + 4 < (int)kHostDiv && a.Kred_pad + bke < kSmallDiv &&
         a.M_total + kWaveRows < kSmallDiv && tiles < kHostDiv && a.R * a.S < (int)kHostDiv && a.H + a.pad < 0x4000 && a.W + a.pad < 0x4000 && a.R < 0x1000 && a.S < 0x1000 && a.stride < 0x1000 &&
         (a.OH - 1) * (double)a.stride < 0x4000 && (a.OW - 1) * (double)a.stride < 0x4000 && a.pad < 0x1000 &&
         a.in_sN >= 0 && a.in_sH >= 0 && a.in_sW >= 0 && ((double)a.N * a.in_sN + a.C) * esz < lim && 128.0 * a.Kred_pad * esz < lim &&
         ((double)a.N * a.out_sN + a.K) * 4 < lim && ((double)a.N * a.res_sN + a.K) * esz < lim;
}
// Do a 3x3 chain's sizes fit the indices of conv3x3_frag_kernel (byte offsets of 32 bits)?
inline bool frag3_takes(const ConvArgs& a) {
  const double lim = 4294967040.0;
  return a.R == 3 && a.S == 3 && a.stride == 1 && a.pad == 1 && a.OH == a.H && a.OW == a.W && a.C % 32 == 0 && a.C >= 32 && a.K % 8 == 0 &&
         a.in_sN >= 0 && a.in_sH >= 0 && a.in_sW >= 0 && ((double)a.N * a.in_sN + a.C) * 2 < lim && ((double)a.N * a.out_sN + a.K) * 2 < lim &&
         ((double)a.N * a.res_sN + a.K) * 2 < lim && (double)((a.K + 127) / 128) * 128 * a.C * 18 < lim;
}
int launch_frag3(const ConvArgs& a, int dtype, void* stream);
int launch_first(const ConvArgs& a, int dtype, void* stream);
// Pixels of the map that the windows of a tile of th x tw depthwise outputs cover, at most
inline int wave_block_positions(const ConvArgs& a, int th, int tw) {
  auto most = [&](int out, int t, int in) {
    int r = 0;
    for (int i = 0; i < out; i += t) r = std::max(r, std::min(i * a.dw_stride + (t - 1) * a.dw_stride + 2, in) - std::max(i * a.dw_stride - 1, 0));
    return r;
  };
  return most(a.OH, th, a.H) * most(a.OW, tw, a.W);
}
// Do a pointwise -> depthwise chain's sizes fit the indices of its wave kernel?
inline bool pwdw_wave_takes(const ConvArgs& a, int esz) {
  const double lim = 2147483648.0, outs = (double)a.N * a.OH * a.OW * std::ceil(a.K / 32.0);   // (a tile is at least one output pixel)
  return a.in_sN >= 0 && a.in_sH >= 0 && a.in_sW >= 0 && ((double)a.N * a.in_sN + a.C) * esz < lim && ((double)a.N * a.out_sN + a.K) * esz < lim &&
         128.0 * a.Kred_pad * esz < lim && outs < kHostDiv && a.Kred_pad * esz / kRowBytes + 4 < (int)kHostDiv;
}
int launch_pwdw_wave(const ConvArgs& a, int dtype, void* stream);
size_t pwdw_wave_lds(const ConvArgs& a, int esz);
constexpr int wave_mid_pitch(int esz) { return 32 * esz + 16; }
int launch_conv_wave(const ConvArgs& a, int dtype, int edge, void* stream);
size_t conv_wave_lds(int edge, int stages, int esz);
int conv_wave_stages(int edge, int steps, int tiles, int esz);   // for shares of `steps` reduction steps of `tiles` tiles
bool conv_cfg_has_scalar_loader(int cfg);
bool conv_cfg_has_dw_prologue(int cfg, int mode);
size_t dwpw_lds_bytes(int panel_channels, int esz);   // LDS of the depthwise-panel kernel for a panel of that many channels
// device probes for the roofline denominators (xenos_kernels.hip)
int launch_probe_mfma(void* d_out, int num_cu, int iters, int data, void* stream, double* flops);
int launch_probe_read(const void* d_in, size_t bytes, void* d_out, int num_cu, void* stream);
size_t probe_out_bytes(int num_cu);
// pointwise -> depthwise kernel (xenos_linked.hip)
int launch_pwdw(const ConvArgs& a, int dtype, void* stream);
size_t pwdw_lds_bytes(int th, int tw, int stride, int esz);
// pointwise -> depthwise -> pointwise kernel (xenos_unit.hip)
int launch_unit(const ConvArgs& a, int dtype, void* stream);
size_t unit_lds_bytes(int th, int tw, int stride, int c1, int c, int esz);
// Fire-module kernel (xenos_linked.hip); conv_h x conv_w = conv-output pixels of a tile
int launch_fire(const ConvArgs& a, int dtype, void* stream);
size_t fire_lds_bytes(int conv_h, int conv_w, int S, int esz, int pooled, int ring = 1);   // ring: halo of the block (1 with a 3x3 part)

}  // namespace xenos
