// Quotients of indices by a run-time integer d from r, an approximation of 1 / d within one unit in the last place (what the
// hardware's reciprocal instruction gives).  Plain arithmetic, the same on the host: tests compile this file by itself.
#pragma once

namespace xenos {

// n / d for 0 <= n < kSmallDiv, exactly: (n + 0.5) / d is at least 0.5 / d away from an integer, and reciprocal, product and
// conversion together are off by less than 2^-21 of it.  Four instructions; the compiler's division by a run-time integer is
// some thirty, several of them at quarter rate, and is what the index arithmetic of a short chain is made of (eight of them in
// the loader of unit_kernel were 3 of the 5 k cycles until its input was in LDS).
constexpr int kSmallDiv = 1 << 20;
__attribute__((always_inline)) constexpr int small_quotient(int n, float r) { return (int)(((float)n + 0.5f) * r); }

// n / d for any 0 <= n < 2^31: the product is off by at most 2^-21 of the quotient, a second one of the remainder leaves at
// most one either way.  Some fifteen instructions.  (Unsigned: a first quotient above the true one times d may reach 2^31.)
__attribute__((always_inline)) constexpr int any_quotient(int n, int d, float r) {
  unsigned q = (unsigned)((float)n * r);
  q += (unsigned)(int)((float)(int)((unsigned)n - q * (unsigned)d) * r);
  const int rem = (int)((unsigned)n - q * (unsigned)d);
  return (int)(rem < 0 ? q - 1 : rem >= d ? q + 1 : q);
}

// n / d for n d < 2^31 by a multiplier that the host has made, one scalar multiplication: the multiplier is less than 1 above 2^31 / d, so that
// 2 n multiplier / 2^32 is n / d and less than n / 2^31 <= 1 / d above it, and n / d is at least 1 / d below the next integer.
constexpr unsigned kHostDiv = 1u << 15;                // (numbers and divisors that need no other look)
__attribute__((always_inline)) constexpr unsigned host_multiplier(unsigned d) { return (unsigned)((0x80000000ull + d - 1) / d); }
__attribute__((always_inline)) constexpr unsigned host_quotient(unsigned n, unsigned mul) { return (unsigned)((2ull * n * mul) >> 32); }
// The multiplier for numbers below `end`: one whose quotients are all 0 where they are, and 0 where there is none
constexpr unsigned host_multiplier(long long end, long long d) {
  return end <= d ? 1u : (end - 1) * d < (1ll << 31) ? host_multiplier((unsigned)d) : 0u;
}

}  // namespace xenos
