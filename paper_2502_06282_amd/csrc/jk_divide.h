// Division by multiplication, for kernels whose divisors are arguments of the call.  Plain C++ (a host test checks it).  Not
// installed.
#pragma once

namespace jk {

// n / d == (n * mg) >> (32 + over) for 0 <= n < bound (below 2^31).  With mg = floor(2^s / d) + 1 = (2^s + e) / d, e <= d, the product is
// n / d and n * e / (d * 2^s), which stays below the next whole number while n * e < 2^s: s is the smallest from 32 on for which
// bound * d <= 2^s.  Then bound * mg <= 2 * bound^2 fits 64 bits.
struct Divisor {
  unsigned long long mg;
  int over;
};
constexpr Divisor divisor(long long bound, int d) {
  int over = 0;
  while (over < 30 && (unsigned long long)bound * (unsigned)d > 1ull << (32 + over)) ++over;
  return Divisor{(1ull << (32 + over)) / (unsigned)d + 1ull, over};
}
constexpr int quotient(int n, unsigned long long mg, int over) { return (int)((unsigned)(((unsigned long long)(unsigned)n * mg) >> 32) >> over); }

// Whether 32 bits of shift are enough
constexpr bool exact_in_32(long long bound, int d) {
  const unsigned long long e = ((1ull << 32) / (unsigned)d + 1ull) * (unsigned)d - (1ull << 32);
  return (unsigned long long)(bound - 1) <= ((1ull << 32) - 1) / e;
}

}  // namespace jk
