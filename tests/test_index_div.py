"""The quotients every kernel index is made of (csrc/index_div.h), on the host: the file itself compiled by the host compiler, with
the reciprocal at its correctly rounded value and one unit in the last place to either side."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2302_00282_amd", "csrc")

PROGRAM = r"""
#include <initializer_list>
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include "index_div.h"
using namespace xenos;

static long long bad = 0, seen = 0;
static void check(int64_t n, int d, bool small_only) {
  if (n < 0 || n > INT32_MAX) return;
  const float r0 = (float)(1.0 / d);
  for (float r : {nextafterf(r0, 0.f), r0, nextafterf(r0, 2.f)}) {
    const int want = (int)(n / d);
    ++seen;
    if (n < kSmallDiv && small_quotient((int)n, r) != want && ++bad < 9) printf("small %lld / %d\n", (long long)n, d);
    if (!small_only && any_quotient((int)n, d, r) != want && ++bad < 9) printf("any %lld / %d\n", (long long)n, d);
  }
}

int main() {
  // every quotient boundary below kSmallDiv of every divisor up to 2048, and of larger ones in growing steps
  for (int64_t d = 1; d < (1ll << 31); d += d < 2048 ? 1 : d / 97 + 1)
    for (int64_t m = 0; m <= kSmallDiv + d; m += d) { check(m - 1, (int)d, true); check(m, (int)d, true); }
  // boundaries over the whole range: around multiples k d with k spread over its octaves, and around the ends of the range
  uint64_t s = 88172645463325252ull;
  for (int64_t d = 1; d < (1ll << 31); d += d < 4096 ? 1 : d / 211 + 1) {
    const int64_t kmax = INT32_MAX / d;
    for (int i = 0; i < 96; ++i) {
      s ^= s << 13; s ^= s >> 7; s ^= s << 17;
      const int64_t k = i < 4 ? kmax - i : (int64_t)(s % (uint64_t)(kmax + 1)) >> (s >> 59);
      for (int o = -1; o <= 1; ++o) check(k * d + o, (int)d, false);
    }
    for (int o = 0; o < 3; ++o) { check(o, (int)d, false); check((int64_t)INT32_MAX - o, (int)d, false); }
  }
  printf("%lld quotients, %lld wrong\n", seen, bad);
  return bad != 0;
}
"""


def test_index_quotients_are_exact_over_their_ranges(tmp_path):
    src, exe = tmp_path / "div.cpp", tmp_path / "div"
    src.write_text(PROGRAM)
    # (float arithmetic as written, signed overflow and conversions out of range are errors)
    subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-fsanitize=signed-integer-overflow,float-cast-overflow",
                    "-fno-sanitize-recover=all", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    print(r.stdout)


HOST_PROGRAM = r"""
#include <initializer_list>
#include <stdint.h>
#include <stdio.h>
#include "index_div.h"
using namespace xenos;

int main() {
  long long bad = 0, seen = 0;
  for (unsigned d = 1; d < kHostDiv; ++d) {
    const unsigned mul = host_multiplier(d);
    auto check = [&](unsigned n) { ++seen; if (n < kHostDiv && host_quotient(n, mul) != n / d && ++bad < 9) printf("host %u / %u\n", n, d); };
    for (unsigned m = 0; m < kHostDiv + d; m += d) { if (m) check(m - 1); check(m); }
    check(kHostDiv - 1);
  }
  // any number whose product with the divisor is below 2^31: every boundary of a divisor, or 200 of them spread evenly and the last, and the ends
  for (int64_t d = 1; d < (1ll << 31); d += d < 70000 ? 1 : d / 211 + 1)
    for (int64_t end : {(int64_t)1, d, d + 1, 3 * d / 2 + 1, (INT32_MAX - d) / d / 3 + 1, INT32_MAX / d + 1}) {
      const unsigned mul = host_multiplier((long long)end, (long long)d);
      const bool none = end > d && (end - 1) * d > INT32_MAX;
      if ((mul == 0) != none && ++bad < 9) printf("multiplier %lld / %lld\n", (long long)end, (long long)d);
      auto check = [&](int64_t n) { ++seen; if (n >= 0 && n < end && n <= INT32_MAX && host_quotient((unsigned)n, mul) != n / d && ++bad < 9) printf("%lld / %lld\n", (long long)n, (long long)d); };
      if (none) continue;
      const int64_t kmax = (end - 1) / d, step = kmax / 200 + 1;
      for (int64_t k = 0; k <= kmax; k += step) { check(k * d - 1); check(k * d); }
      for (int64_t n : {kmax * d - 1, kmax * d, end - 2, end - 1}) check(n);
    }
  printf("%lld quotients, %lld wrong\n", seen, bad);
  return bad != 0;
}
"""


def test_quotients_by_host_made_multipliers_are_exact(tmp_path):
    # every quotient boundary of every divisor in the range
    src, exe = tmp_path / "host.cpp", tmp_path / "host"
    src.write_text(HOST_PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
