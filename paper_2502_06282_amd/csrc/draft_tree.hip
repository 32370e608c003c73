// Growing the draft token tree on the device (gfx950), one depth at a time, from the candidate
// lists that jk_draft_heads returns (Section 3.1.2 of the paper: both activated experts propose
// their own top-k candidates for every expanded node, the expert with the larger router score
// on the left; top-k construction as in a dynamically built tree).
//
//   grow      per sequence: a new node for every (frontier node, expert, rank) in that order,
//             score = parent's score * candidate probability; the `width` best new nodes (ties
//             to the lower index) become the next frontier, listed in increasing index.
//   finalize  per sequence: the n_keep best nodes (ties to the lower index; a node never scores
//             above its parent, so ancestors come along), renumbered in increasing old index.
//   gather    the kept nodes' draft distributions as the dense [batch][n_tree][vocab] array that
//             jk_accept_path takes.
// Choices are made by counting how many entries beat a given one (no sorting network, no reduction rounds), among a few hundred
// entries per sequence: where more are cut, among those in the bin of scores that the last kept one lies in.
#include <climits>

#include "jk_internal.h"
#include "jk_wave.h"

namespace jk {
namespace {

constexpr int kTreeThreads = 256;
constexpr int kTreeWaves = kTreeThreads / 64;
constexpr int kMaxGrowNodes = 1024;  // node capacity per sequence the kernels are laid out for

typedef float floatx4 __attribute__((ext_vector_type(4)));

// larger score first, equal scores by increasing index (both operands always evaluated)
__device__ __forceinline__ int beats(float av, int ai, float bv, int bi) {
  return (int)(av > bv) | ((int)(av == bv) & (int)(ai < bi));
}

// s_rank[i] += how many of the n entries of s_sc beat entry i; s_sc holds -inf from n to the next multiple of four (an
// index beyond n never wins a tie), s_rank starts at zero, and a barrier on either side is the caller's.  A wave takes
// 64 entries i and a part of the entries j that they are held against: a few entries still occupy every wave (one wave
// for 50 candidates spent as long comparing as a trip to memory takes).  Whether j or i is lower is known for all but
// the wave's own 64 entries, and one comparison is enough there.
template <int kWaves>
__device__ __forceinline__ void count_beaten(const float* s_sc, int n, int* s_rank, int t) {
  const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int chunks = (n + 63) >> 6, parts = chunks >= kWaves ? 1 : kWaves / max(chunks, 1);
  const int len = ((n + parts - 1) / parts + 3) & ~3;
  for (int u = wave; u < chunks * parts; u += kWaves) {
    const int c0 = (u / parts) * 64, p = u - (u / parts) * parts;
    const int j0 = p * len, j1 = min(j0 + len, (n + 3) & ~3);
    const int i = c0 + lane;
    const float sc = s_sc[min(i, n - 1)];
    int rank = 0, j = j0;
#pragma unroll 4
    for (; j < min(j1, c0); j += 4) {
      const floatx4 v = *reinterpret_cast<const floatx4*>(s_sc + j);
      rank += (int)(v[0] >= sc) + (int)(v[1] >= sc) + (int)(v[2] >= sc) + (int)(v[3] >= sc);
    }
#pragma unroll 4
    for (; j < min(j1, c0 + 64); j += 4) {
      const floatx4 v = *reinterpret_cast<const floatx4*>(s_sc + j);
      rank += beats(v[0], j, sc, i) + beats(v[1], j + 1, sc, i) + beats(v[2], j + 2, sc, i) + beats(v[3], j + 3, sc, i);
    }
#pragma unroll 4
    for (; j < j1; j += 4) {
      const floatx4 v = *reinterpret_cast<const floatx4*>(s_sc + j);
      rank += (int)(v[0] > sc) + (int)(v[1] > sc) + (int)(v[2] > sc) + (int)(v[3] > sc);
    }
    if (i < n) atomicAdd(&s_rank[i], rank);
  }
}

// How many threads with a smaller index raised `flag`, and how many did in all: ballots within the waves, the waves'
// totals through LDS (s_cnt: kWaves ints; the caller's later use of it must follow a barrier).
template <int kWaves>
__device__ __forceinline__ int count_before(bool flag, int t, int* s_cnt, int& total) {
  const unsigned long long m = __ballot(flag);
  const int lane = t & 63, wave = t >> 6;
  const int in_wave = __popcll(m & ((1ull << lane) - 1ull));
  if (lane == 0) s_cnt[wave] = __popcll(m);
  __syncthreads();
  int before = in_wave;
  total = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const int c = s_cnt[w];
    before += w < wave ? c : 0;
    total += c;
  }
  return before;
}

// Bound by latency: a few hundred bytes per sequence, so what counts is how many trips to memory follow each other, and
// behind them the instructions of a wave (8 cycles each where one waits for the other).  Everything is asked for at once: the
// candidate, its token, the frontier entry, the node count, and the scores of all nodes, of which the parents' are then taken
// from LDS instead of memory.  Four waves for each 64 candidates hold them against each other.  us under the tracer, eight
// sequences, the parent's score asked for behind the frontier's entry and four waves for any number / like this: five expanded
// nodes of ten candidates 3.8 / 3.7, ten of 18 6.2 / 5.1.
template <int kWaves>
__global__ __launch_bounds__(64 * kWaves) void grow_kernel(TreeGrowArgs a) {
  constexpr int kThreads = 64 * kWaves, kOld = kMaxGrowNodes / kThreads;
  __shared__ __align__(16) float s_sc[kTreeThreads];
  __shared__ float s_old[kMaxGrowNodes];
  __shared__ int s_rank[kTreeThreads];
  __shared__ int s_cnt[kWaves];
  __shared__ int s_first;
  const int b = blockIdx.x, t = threadIdx.x;
  const int C = a.n_front * 2 * a.top_k;  // <= kTreeThreads (checked by the host)
  const int slot_e = (int)(((unsigned)min(t, C - 1) * a.mg_top_k) >> 16);  // candidate / top_k
  const int f = slot_e >> 1, e = slot_e & 1;
  const long long row = (long long)b * a.n_front + f, at_c = (long long)b * C + min(t, C - 1), first = (long long)b * a.max_nodes;
  const int n_raw = a.n_nodes[b];
  const float p = a.cand_p[at_c];
  const int tok = a.cand_tok[at_c];
  int pid = -1;
  float old_score[kOld];
  if (a.frontier_in) {
    pid = a.frontier_in[row];
#pragma unroll
    for (int i = 0; i < kOld; ++i) old_score[i] = a.score[first + min(t + kThreads * i, a.max_nodes - 1)];
#pragma unroll
    for (int i = 0; i < kOld; ++i) s_old[t + kThreads * i] = old_score[i];
  }
  if (t < kTreeThreads) s_rank[t] = 0;
  if (t == 0) s_first = INT_MAX;
  __syncthreads();
  const int n0 = min(max(n_raw, 0), a.max_nodes);  // (a count the caller forgot to clear must not fault)
  const int id = n0 + t;
  const bool valid = t < C && id < a.max_nodes;
  const bool old = pid >= 0 && pid < n0;
  const float sc = valid ? (old ? s_old[pid] : 1.0f) * p : -INFINITY;
  if (t < kTreeThreads) s_sc[t] = sc;  // (entries from C on hold -inf and a larger index: they beat nobody)
  if (valid) {
    const long long at = first + id;
    a.tokens[at] = tok;
    a.parent[at] = old ? pid : -1;
    a.score[at] = sc;
    a.q_row[at] = a.q_row_base + (int)(2 * row) + e;
  }
  __syncthreads();
  count_beaten<kWaves>(s_sc, C, s_rank, t);
  __syncthreads();
  const bool sel = valid && s_rank[t] < a.width;
  int total;
  const int slot = count_before<kWaves>(sel, t, s_cnt, total);
  if (sel) {
    a.frontier_out[(long long)b * a.width + slot] = id;
    if (slot == 0) s_first = id;
  }
  if (total < a.width) {  // (uniform) fewer new nodes than frontier slots: the rest repeats the first entry (-1 if there is none)
    __syncthreads();
    if (t >= total && t < a.width) a.frontier_out[(long long)b * a.width + t] = s_first == INT_MAX ? -1 : s_first;
  }
  if (t == 0) a.n_nodes[b] = min(n0 + C, a.max_nodes);
}

// The last draft pass with a mixture head and a contrastive head (Section 3.2): children from
// head 0's list, then the `width` best children get head 1's list of their parent as children.
__global__ __launch_bounds__(kTreeThreads) void grow_tail_kernel(TreeGrowArgs a, int k1, int k2) {
  __shared__ __align__(16) float s_sc[kTreeThreads];
  __shared__ int s_rank[kTreeThreads];
  __shared__ int s_cnt[kTreeWaves];
  __shared__ int s_child[kTreeThreads];  // chosen children by slot: node id, frontier slot
  __shared__ int s_slot_f[kTreeThreads];
  const int b = blockIdx.x, t = threadIdx.x;
  const int C = a.n_front * k1;
  const int n0 = min(max(a.n_nodes[b], 0), a.max_nodes);
  const int id = n0 + t;
  const bool valid = t < C && id < a.max_nodes;
  const long long base = (long long)b * a.max_nodes;
  float sc = -INFINITY;
  const int f = t / k1, j = t - f * k1;
  if (valid) {
    const long long row = (long long)b * a.n_front + f;
    const int pid = a.frontier_in ? a.frontier_in[row] : -1;
    const bool has_parent = pid >= 0 && pid < n0;
    const float ps = has_parent ? a.score[base + pid] : 1.0f;
    sc = ps * a.cand_p[row * 2 * a.top_k + j];
    a.tokens[base + id] = a.cand_tok[row * 2 * a.top_k + j];
    a.parent[base + id] = has_parent ? pid : -1;
    a.score[base + id] = sc;
    a.q_row[base + id] = a.q_row_base + (int)(2 * row);
  }
  s_sc[t] = sc;
  s_rank[t] = 0;
  __syncthreads();
  count_beaten<kTreeWaves>(s_sc, C, s_rank, t);
  __syncthreads();
  const bool sel = valid && s_rank[t] < a.width;
  int total;
  const int slot = count_before<kTreeWaves>(sel, t, s_cnt, total);
  if (sel) {
    s_child[slot] = id;
    s_slot_f[slot] = f;
  }
  __syncthreads();
  const int n1 = min(n0 + C, a.max_nodes);
  const int G = total * k2;
  const int gid = n1 + t;
  if (t < G && gid < a.max_nodes) {
    const int s = t / k2, j2 = t - s * k2;
    const int c = s_child[s];
    const long long row = (long long)b * a.n_front + s_slot_f[s];
    a.tokens[base + gid] = a.cand_tok[(row * 2 + 1) * a.top_k + j2];
    a.parent[base + gid] = c;
    a.score[base + gid] = s_sc[c - n0] * a.cand_p[(row * 2 + 1) * a.top_k + j2];
    a.q_row[base + gid] = a.q_row_base + (int)(2 * row) + 1;
  }
  if (t == 0) a.n_nodes[b] = min(n1 + G, a.max_nodes);
}

// One depth of a predefined tree shape: new node j hangs under frontier slot shape_slot[j] and
// takes candidate shape_rank[j] of that slot's list of expert shape_expert[j].
__global__ __launch_bounds__(kTreeThreads) void fill_static_kernel(TreeGrowArgs a, const int* __restrict__ shape_slot,
                                                                   const int* __restrict__ shape_expert,
                                                                   const int* __restrict__ shape_rank, int n_new,
                                                                   const int* __restrict__ next_index, int n_next,
                                                                   int* __restrict__ new_ids) {
  const int b = blockIdx.x, t = threadIdx.x;
  const int n0 = min(max(a.n_nodes[b], 0), a.max_nodes);
  const long long base = (long long)b * a.max_nodes;
  for (int j = t; j < n_new; j += kTreeThreads) {
    const int id = n0 + j;
    const bool valid = id < a.max_nodes;
    if (valid) {
      const int f = min(max(shape_slot[j], 0), a.n_front - 1);
      const int e = shape_expert[j] != 0 ? 1 : 0;
      const int r = min(max(shape_rank[j], 0), a.top_k - 1);
      const long long row = (long long)b * a.n_front + f;
      const int pid = a.frontier_in ? a.frontier_in[row] : -1;
      const bool has_parent = pid >= 0 && pid < n0;
      const float ps = has_parent ? a.score[base + pid] : 1.0f;
      a.tokens[base + id] = a.cand_tok[(row * 2 + e) * a.top_k + r];
      a.parent[base + id] = has_parent ? pid : -1;
      a.score[base + id] = ps * a.cand_p[(row * 2 + e) * a.top_k + r];
      a.q_row[base + id] = a.q_row_base + (int)(2 * row) + e;
    }
    if (new_ids) new_ids[(long long)b * n_new + j] = valid ? id : -1;
  }
  if (a.frontier_out)
    for (int i = t; i < n_next; i += kTreeThreads) {
      const int j = min(max(next_index[i], 0), n_new - 1);
      a.frontier_out[(long long)b * n_next + i] = n0 + j < a.max_nodes ? n0 + j : -1;
    }
  __syncthreads();  // everybody has read n_nodes
  if (t == 0) a.n_nodes[b] = min(n0 + n_new, a.max_nodes);
}

// Order of scores as unsigned numbers (the two zeros are equal; a NaN's key is not used)
__device__ __forceinline__ unsigned score_key(float v) {
  const unsigned u = __float_as_uint(v + 0.f);
  return (u >> 31) ? ~u : u | 0x80000000u;
}

// A thread per node.  Everything a node holds is asked for before its sequence's node count is known (the arrays are
// max_nodes long): one trip to memory instead of three.  Which nodes are kept: a histogram of the scores' upper bits (sign,
// exponent and two more: some five nodes to a bin) says in which bin the last one lies; the nodes of that bin alone are held
// against each other.  us under the tracer, eight sequences, every node held against every other / like this: 260 nodes 6.4 / 5.2, 1020 nodes
// 21.6 / 8.4 (and 18.2 for 260 with four waves and three trips).
__global__ __launch_bounds__(kMaxGrowNodes) void finalize_kernel(TreeFinalArgs a) {
  constexpr int kWaves = kMaxGrowNodes / 64, kBins = 2 * kMaxGrowNodes;
  static_assert(kBins == 2048, "eleven bits");
  __shared__ __align__(16) int s_bins[kBins];
  __shared__ unsigned s_key[kMaxGrowNodes];  // of the nodes in the last bin, and who they are
  __shared__ short s_who[kMaxGrowNodes];
  __shared__ short s_new[kMaxGrowNodes];
  __shared__ int s_cnt[kWaves], s_above[kWaves];
  __shared__ int s_bin, s_need, s_members;
  const int b = blockIdx.x, t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const long long at = (long long)b * a.max_nodes + min(t, a.max_nodes - 1);
  const int n_raw = a.n_nodes[b];
  const float sc = a.score[at];
  const int pid = a.parent[at], tok = a.tokens[at], q_row = a.q_row[at];
  *reinterpret_cast<int2*>(s_bins + 2 * t) = make_int2(0, 0);
  if (t == 0) {
    s_bin = -1;  // (as many nodes as are wanted, or fewer: all of them)
    s_need = 0;
    s_members = 0;
  }
  __syncthreads();
  const int n = min(max(n_raw, 0), a.max_nodes);
  const bool real = t < n, ranked = real && sc == sc;  // (a NaN is beaten by nobody and beats nobody)
  const unsigned key = score_key(sc);
  const int bin = (int)(key >> 21);
  if (ranked) atomicAdd(&s_bins[bin], 1);
  __syncthreads();
  {  // a thread has two bins, the highest first: the nodes in front of its own
    const int2 mine = *reinterpret_cast<const int2*>(s_bins + kBins - 2 - 2 * t);
    const int sum = mine.x + mine.y, upto = dev::wave_scan(sum);
    if (lane == 63) s_above[wave] = upto;
    __syncthreads();
    int before = upto - sum;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) before += w < wave ? s_above[w] : 0;
    if (before < a.n_keep && before + mine.y >= a.n_keep) {
      s_bin = kBins - 1 - 2 * t;
      s_need = a.n_keep - before;
    }
    before += mine.y;
    if (before < a.n_keep && before + mine.x >= a.n_keep) {
      s_bin = kBins - 2 - 2 * t;
      s_need = a.n_keep - before;
    }
  }
  __syncthreads();
  const int last = s_bin, need = s_need;
  bool kept = real && (!ranked || bin > last);
  const bool member = ranked && bin == last;
  if (member) {
    const int i = atomicAdd(&s_members, 1);
    s_key[i] = key;
    s_who[i] = (short)t;
  }
  __syncthreads();
  if (member) {
    const int members = s_members;
    int rank = 0;
#pragma unroll 4
    for (int i = 0; i < members; ++i) {
      const unsigned other = s_key[i];
      rank += (int)(other > key) | ((int)(other == key) & (int)(s_who[i] < t));
    }
    kept = rank < need;
  }
  int total;
  const int place = count_before<kWaves>(kept, t, s_cnt, total);
  s_new[t] = (short)place;
  __syncthreads();
  if (kept && place < a.n_keep) {
    const long long o = (long long)b * a.n_keep + place;
    a.out_tokens[o] = tok;
    a.out_parent[o] = (pid >= 0 && pid < t) ? (int)s_new[pid] : -1;  // (a kept node's parent is kept)
    a.out_q_row[o] = q_row;
    if (a.out_old) a.out_old[o] = t;
  }
  const int n_valid = min(n, a.n_keep);
  for (int i = n_valid + t; i < a.n_keep; i += kMaxGrowNodes) {  // a tree with fewer nodes than asked for
    const long long o = (long long)b * a.n_keep + i;
    a.out_tokens[o] = -1;
    a.out_parent[o] = -1;
    a.out_q_row[o] = 0;
    if (a.out_old) a.out_old[o] = -1;
  }
  if (t == 0) a.n_valid[b] = n_valid;
}

__global__ __launch_bounds__(256) void reset_kernel(int32_t* n_nodes, int batch) {
  const int b = blockIdx.x * 256 + threadIdx.x;
  if (b < batch) n_nodes[b] = 0;
}

__global__ __launch_bounds__(256) void gather_rows_kernel(const float* __restrict__ q_all, const int* __restrict__ q_row,
                                                          float* __restrict__ out, int vocab, long long n_q_rows) {
  const long long node = blockIdx.x;
  long long r = q_row[node];
  r = r < 0 ? 0 : (r >= n_q_rows ? n_q_rows - 1 : r);  // must not fault on a bad row number
  const float* src = q_all + r * vocab;
  float* dst = out + node * vocab;
  const bool vec = (vocab & 3) == 0 && ((reinterpret_cast<size_t>(q_all) | reinterpret_cast<size_t>(out)) & 15) == 0;
  if (vec) {
    for (int c = blockIdx.y * 256 + threadIdx.x; c < vocab / 4; c += 256 * gridDim.y)
      reinterpret_cast<floatx4*>(dst)[c] = reinterpret_cast<const floatx4*>(src)[c];
  } else {
    for (int c = blockIdx.y * 256 + threadIdx.x; c < vocab; c += 256 * gridDim.y) dst[c] = src[c];
  }
}

}  // namespace

int tree_max_nodes() { return kMaxGrowNodes; }

hipError_t launch_tree_grow(const TreeGrowArgs& a, hipStream_t stream) {
  // Four waves for each 64 candidates (the state's stores and loads take 256 threads whatever their number)
  const int chunks = (a.n_front * 2 * a.top_k + 63) / 64;
  if (chunks <= 1) return launch_kernel(grow_kernel<4>, dim3(a.batch), dim3(256), 0, stream, a);
  if (chunks == 2) return launch_kernel(grow_kernel<8>, dim3(a.batch), dim3(512), 0, stream, a);
  return launch_kernel(grow_kernel<16>, dim3(a.batch), dim3(1024), 0, stream, a);
}
hipError_t launch_tree_grow_tail(const TreeGrowArgs& a, int k1, int k2, hipStream_t stream) {
  return launch_kernel(grow_tail_kernel, dim3(a.batch), dim3(kTreeThreads), 0, stream, a, k1, k2);
}
hipError_t launch_tree_fill_static(const TreeGrowArgs& a, const int* slot, const int* expert, const int* rank, int n_new,
                                   const int* next_index, int n_next, int* new_ids, hipStream_t stream) {
  return launch_kernel(fill_static_kernel, dim3(a.batch), dim3(kTreeThreads), 0, stream, a, slot, expert, rank, n_new, next_index, n_next, new_ids);
}
hipError_t launch_tree_finalize(const TreeFinalArgs& a, hipStream_t stream) {
  return launch_kernel(finalize_kernel, dim3(a.batch), dim3(kMaxGrowNodes), 0, stream, a);
}
hipError_t launch_tree_reset(int32_t* n_nodes, int batch, hipStream_t stream) {
  return launch_kernel(reset_kernel, dim3(((unsigned)batch + 255u) / 256u), dim3(256), 0, stream, n_nodes, batch);
}
hipError_t launch_gather_rows(const float* q_all, const int* q_row, float* out, long long n_nodes, int vocab,
                              long long n_q_rows, hipStream_t stream) {
  const unsigned chunks = (unsigned)(vocab / 4096 < 1 ? 1 : (vocab / 4096 > 16 ? 16 : vocab / 4096));
  hipLaunchKernelGGL(gather_rows_kernel, dim3((unsigned)n_nodes, chunks), dim3(256), 0, stream, q_all, q_row, out,
                     vocab, n_q_rows);
  return hipGetLastError();
}

}  // namespace jk
