// The ancestors of a tree's nodes, made by a wave in its registers (gfx950).  Not installed.
#pragma once
#include "jk_internal.h"

namespace jk {
namespace dev {

// The ancestors of a node (with itself), as a lane needs them for its row: bits of nodes 0 - 63 and 64 - 127.  A lane holds
// nodes lane and lane + 64; sets and pointers double their reach every round, by exchanges across the wave: no barrier, and no
// wave that the others wait for.  (One wave for all, through LDS: it came 2500 cycles after the others to the barrier.)
struct Ancestors {
  unsigned long long lo, hi;
};
__device__ __forceinline__ unsigned long long shfl64(unsigned long long v, int lane) {
  return (unsigned)__shfl((int)(unsigned)v, lane) | (unsigned long long)(unsigned)__shfl((int)(unsigned)(v >> 32), lane) << 32;
}
// pa0, pa1: parents of nodes lane and lane + 64.  An entry that is no parent counts as -1; `report`: into the error word
__device__ __forceinline__ Ancestors ancestors_of(int T, unsigned* err, int pa0, int pa1, int node, bool report) {
  const int lane = threadIdx.x & 63;
  const bool ok0 = lane >= T || (pa0 >= -1 && pa0 < lane), ok1 = lane + 64 >= T || (pa1 >= -1 && pa1 < lane + 64);
  if (report && __any(!ok0 || !ok1) && lane == 0) __hip_atomic_fetch_or(err, kDevErrBadTree, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  int up0 = ok0 && lane < T ? pa0 : -1;
  unsigned long long own0 = 1ull << lane;  // of node `lane`: all its ancestors are below 64
  while (__any(up0 >= 0)) {
    const int from = max(up0, 0);
    const unsigned long long set = shfl64(own0, from);
    const int next = __shfl(up0, from);
    if (up0 >= 0) {
      own0 |= set;
      up0 = next;
    }
  }
  if (T <= 64) return Ancestors{shfl64(own0, node), 0ull};
  int up1 = ok1 && lane + 64 < T ? pa1 : -1;
  unsigned long long low1 = 0ull, own1 = 1ull << lane;  // of node lane + 64
  while (__any(up1 >= 0)) {
    const int from = max(up1, 0) & 63;
    const unsigned long long below = shfl64(own0, from), low = shfl64(low1, from), set = shfl64(own1, from);
    const int next = __shfl(up1, from);
    if (up1 >= 64) {
      low1 |= low;
      own1 |= set;
      up1 = next;
    } else if (up1 >= 0) {
      low1 |= below;
      up1 = -1;
    }
  }
  const unsigned long long a = shfl64(own0, node & 63), l = shfl64(low1, node & 63), h = shfl64(own1, node & 63);
  return node < 64 ? Ancestors{a, 0ull} : Ancestors{l, h};
}

}  // namespace dev
}  // namespace jk
