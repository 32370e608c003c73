// csrc/jk_divide.h against division: around the multiples of a divisor, near the ends of a range, for divisors and bounds of every size.
#include <cstdio>
#include <initializer_list>
#include <random>

#include "jk_divide.h"

int main() {
  std::mt19937_64 rng(1);
  long long bad = 0, checked = 0, more = 0, narrow_wrong = 0;
  auto check = [&](long long bound, int d) {
    if (bound < 1 || bound > 0x7fffffffLL || d < 1) return;
    const jk::Divisor by = jk::divisor(bound, d);
    const bool in_32 = jk::exact_in_32(bound, d);
    const unsigned long long mg32 = (1ull << 32) / (unsigned)d + 1ull;
    more += by.over > 0;
    bool narrow = true;
    auto one = [&](long long n) {
      if (n < 0 || n >= bound) return;
      ++checked;
      bad += jk::quotient((int)n, by.mg, by.over) != n / d;
      narrow = narrow && (int)(((unsigned long long)n * mg32) >> 32) == n / d;
    };
    for (long long n : {0LL, 1LL, bound - 1, bound - 2}) one(n);
    for (int i = 0; i < 40; ++i) {
      const long long k = i < 8 ? bound / d - i : (long long)(rng() % (unsigned long long)(bound / d + 1));
      one(k * d - 1);
      one(k * d);
      one(k * d + 1);
    }
    if (in_32 && !narrow) ++bad;  // (said to be exact, and is not)
    if (bound % d == 0) {         // (then it says exactly when it is: the last number is the first to go wrong)
      bad += in_32 != narrow;
      narrow_wrong += !narrow;
    }
  };
  for (int nodes : {1, 2, 60, 128})
    for (int d : {1, 2, 3, 7, 8, 4095, 4096, 5792, 5793, 6000, 8191, 8192, 65535, 65536, 65537, 1 << 20, (1 << 24) - 1}) check((long long)nodes * d, d);
  for (int i = 0; i < 200000; ++i) {
    const int d = 1 + (int)(rng() >> (33 + rng() % 31));
    check(1 + (long long)(rng() >> (33 + rng() % 31)), d);
    check((long long)d * (1 + (int)(rng() % 128)), d);
  }
  std::printf("%lld of %lld wrong; %lld with more than 32 bits, %lld that 32 would get wrong\n", bad, checked, more, narrow_wrong);
  return bad == 0 && more > 0 && narrow_wrong > 0 ? 0 : 1;
}
