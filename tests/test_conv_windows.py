"""The 32-bit windows of conv_kernel's loader for reductions whose tap is uniform (csrc/kernels.h), on the host: what conv_tile_span
says against every offset that the tiles of small chains reach, in each order in which a tile enumerates its pixels."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2302_00282_amd", "csrc")

PROGRAM = r"""
#include <stdio.h>
#include <string.h>
#include "kernels.h"
using namespace xenos;

static uint64_t s = 88172645463325252ull;
static int draw(int lo, int hi) {
  s ^= s << 13; s ^= s >> 7; s ^= s << 17;
  return lo + (int)(s % (uint64_t)(hi - lo + 1));
}

int main() {
  long long bad = 0, seen = 0;
  double tightest = 1e9;
  for (int trial = 0; trial < 20000; ++trial) {
    ConvArgs a;
    memset(&a, 0, sizeof a);
    a.N = draw(1, 5); a.H = draw(1, 40); a.W = draw(1, trial % 4 ? 24 : 300); a.C = draw(1, 4);
    a.R = draw(1, 5); a.S = draw(1, 5); a.stride = draw(1, 3); a.pad = draw(0, 2);
    if (a.H + 2 * a.pad < a.R || a.W + 2 * a.pad < a.S) continue;
    a.OH = (a.H + 2 * a.pad - a.R) / a.stride + 1; a.OW = (a.W + 2 * a.pad - a.S) / a.stride + 1;
    a.in_sW = a.C + draw(0, 3); a.in_sH = a.W * a.in_sW; a.in_sN = a.H * a.in_sH + draw(0, 1) * draw(0, 2000);
    static const int modes[] = {M_FLAT, M_ZIGZAG, M_PATCH, M_GAP};
    a.mode = modes[trial / 7 % 4];
    a.PH = a.OH; a.PW = a.OW;
    if (a.mode == M_ZIGZAG) { a.PH = a.OH / 2; a.PW = a.OW / 2; if (!a.PH || !a.PW) continue; }
    const int BM = 32 << draw(0, 2), pw = draw(1, BM), ph = BM / pw;
    const int total = a.mode == M_FLAT ? a.N * a.OH * a.OW : a.mode == M_ZIGZAG ? a.N * a.PH * a.PW * 4 : a.mode == M_GAP ? a.OH * a.OW : ph * pw;
    const int images = a.mode == M_FLAT || a.mode == M_ZIGZAG ? 1 : a.N;
    const double span = conv_tile_span(a, 1);
    for (int img = 0; img < images; ++img)
      for (int patch = 0; patch < (a.mode == M_PATCH ? 6 : 1); ++patch) {
        const int oy0 = a.mode == M_PATCH ? draw(-2, a.OH) : 0, ox0 = a.mode == M_PATCH ? draw(-2, a.OW) : 0;
        for (int m0 = 0; m0 < total; m0 += BM)
          for (int first = 0; first < BM; first += 8) {              // a wavefront's first row
            int n_first = 0, ih_first = 0;
            for (int row = first; row < BM; ++row) {
              const int m = m0 + row;
              int n = img, oh, ow;
              bool ok = m < total;
              if (a.mode == M_FLAT) { n = m / (a.OH * a.OW); const int p = m % (a.OH * a.OW); oh = p / a.OW; ow = p % a.OW; }
              else if (a.mode == M_ZIGZAG) {
                const int w = m >> 2, q = w % (a.PH * a.PW);
                n = w / (a.PH * a.PW); oh = 2 * (q / a.PW) + ((m & 3) >> 1); ow = 2 * (q % a.PW) + (m & 1);
              } else if (a.mode == M_PATCH) { oh = oy0 + row / pw; ow = ox0 + row % pw; ok = row / pw < ph && oh >= 0 && oh < a.OH && ow >= 0 && ow < a.OW; }
              else { oh = m / a.OW; ow = m % a.OW; }
              const int ih0 = oh * a.stride - a.pad, iw0 = ow * a.stride - a.pad;
              if (row == first) { n_first = n; ih_first = ih0 < 0 ? 0 : ih0 < a.H ? ih0 : a.H; }
              if (!ok) continue;
              for (int r = 0; r < a.R; ++r)
                for (int c = 0; c < a.S; c += a.S > 1 ? a.S - 1 : 1) {
                  const int ih = ih0 + r, iw = iw0 + c;
                  if (ih < 0 || ih >= a.H || iw < 0 || iw >= a.W) continue;
                  const long long off = (n - n_first) * a.in_sN + (ih - ih_first) * a.in_sH + iw * a.in_sW;
                  ++seen;
                  if (off < 0 || off + a.C > span) { if (++bad < 9) printf("mode %d off %lld span %.0f\n", a.mode, off, span); }
                  else if (span / (off + a.C) < tightest) tightest = span / (off + a.C);
                }
            }
          }
      }
  }
  printf("%lld offsets, %lld outside, tightest %.2f\n", seen, bad, tightest);
  ConvArgs b;                                                        // one image or two of 16 GB in rows of 1 MB: a tile sees a few rows
  memset(&b, 0, sizeof b);
  b.mode = M_FLAT; b.H = b.OH = 1 << 14; b.W = b.OW = 1 << 12; b.C = 64; b.R = b.S = 3; b.stride = 1; b.pad = 1; b.Kred_pad = 576;
  b.in_sW = 64; b.in_sH = 64ll << 12; b.in_sN = b.in_sH << 14;
  for (b.N = 1; b.N <= 2; ++b.N)
    if (!conv_window_fits(b, 4)) { ++bad; printf("large image\n"); }
  b.in_sH <<= 10; b.W <<= 10; b.in_sN <<= 10;                        // rows of 1 GB do not fit
  if (conv_window_fits(b, 4)) { ++bad; printf("large rows\n"); }
  return bad != 0 || tightest > 1.2;
}
"""


def test_a_tile_reads_nothing_outside_its_window(tmp_path):
    src, exe = tmp_path / "w.cpp", tmp_path / "w"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
