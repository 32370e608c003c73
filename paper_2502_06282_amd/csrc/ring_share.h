// How the workgroups of ring_gemm.hip divide the groups of weight rows and go through them, apart from what is done with a
// group: the kernel walks this with its own steps, and a host test with steps that check it.  Not installed.
#pragma once

namespace jk {
namespace ring {

// Groups off .. off + size - 1 of an item (an expert with some of the rows that chose it; the output heads are one item)
struct Batch {
  int item, off, size;
};

// The groups of all items, `per_item` each, one item's behind the other's; workgroup `id` of `all` has an equal share, from
// share_begin(id) up to share_begin(id + 1), and goes through it in batches of up to `most` groups of one item.
struct Shares {
  int per_item, most;
  constexpr unsigned share_begin(int items, int id, int all) const {  // (at most 96 x 8192 groups, heads 2^20; all <= 1024)
    return (unsigned)items * (unsigned)per_item * (unsigned)id / (unsigned)all;
  }
  constexpr Batch at(int item, int off, int left) const {  // as even as they come; left > 0: groups of the share from here on
    const int here = per_item - off < left ? per_item - off : left, n = (here + most - 1) / most;
    return Batch{item, off, (here + n - 1) / n};
  }
  constexpr Batch first(int begin, int end) const {  // of a share that is not empty
    const int item = begin / per_item;
    return at(item, begin - item * per_item, end - begin);
  }
  constexpr Batch next(const Batch& b, int left) const {  // left > 0, without b
    const int off = b.off + b.size;
    return off < per_item ? at(b.item, off, left) : at(b.item + 1, 0, left);
  }
};

}  // namespace ring
}  // namespace jk
