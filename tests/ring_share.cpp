// Walks the shares of csrc/ring_share.h as the kernel does: every group of every item comes exactly once, in order, in batches
// of at least one and at most `most` groups that stay within an item and differ by no more than one where an item is divided.
#include <cstdio>
#include <initializer_list>

#include "ring_share.h"

namespace {
int walk(int items, int per_item, int most, int all) {
  const jk::ring::Shares s{per_item, most};
  unsigned seen = 0;
  for (int id = 0; id < all; ++id) {
    const int f0 = (int)s.share_begin(items, id, all), f1 = (int)s.share_begin(items, id + 1, all);
    if ((unsigned)f0 != seen || f1 < f0 || f1 - f0 > ((long long)items * per_item + all - 1) / all) return 1;
    if (f0 == f1) continue;
    jk::ring::Batch b = s.first(f0, f1);
    int smallest = most, largest = 0;
    for (int left = f1 - f0;;) {
      if (b.size < 1 || b.size > most || b.size > left || b.item < 0 || b.item >= items || b.off < 0 || b.off + b.size > per_item) return 2;
      if ((unsigned)(b.item * per_item + b.off) != seen) return 3;
      seen += (unsigned)b.size;
      smallest = b.size < smallest ? b.size : smallest;
      largest = b.size > largest ? b.size : largest;
      if ((left -= b.size) <= 0) break;
      b = s.next(b, left);
    }
    if (items == 1 && largest - smallest > 1) return 4;
  }
  return seen == (unsigned)items * (unsigned)per_item ? 0 : 5;
}
}  // namespace

int main() {
  const int per[] = {1, 2, 3, 5, 7, 16, 17, 31, 64, 255, 256, 257, 511, 8192};
  const int all[] = {1, 2, 7, 8, 255, 256, 304, 1024};
  long long walks = 0;
  for (int most : {2, 4, 6})
    for (int a : all) {
      for (int items : {0, 1, 2, 3, 5, 8, 63, 64, 96})
        for (int p : per) {
          ++walks;
          if (const int bad = walk(items, p, most, a)) return std::printf("%d items of %d, batches of %d, %d workgroups: %d\n", items, p, most, a, bad), 1;
        }
      for (int p = 513; p < (1 << 20); p = p * 3 + 1) {
        ++walks;
        if (const int bad = walk(1, p, most, a)) return std::printf("%d groups, batches of %d, %d workgroups: %d\n", p, most, a, bad), 1;
      }
      if (const int bad = walk(1, 1 << 20, most, a)) return std::printf("2^20 groups: %d\n", bad), 1;
    }
  std::printf("%lld walks\n", walks);
  return 0;
}
