// The sampling walk of one tree by one workgroup: waits for nobody.  walk_sample_kernel (accept.hip) is this for every tree;
// walk_sample_wide_kernel (accept_coop.hip) falls back on it where the workgroups of a tree did not meet.  Not installed.
#pragma once
#include "jk_internal.h"

namespace jk {
namespace dev {

// A parent entry that breaks -1 <= parent[k] < k counts as -1, and a token id outside the vocabulary is
// clamped into it; either is recorded in the workspace's sticky error word (err may be null).
__device__ __forceinline__ void report(unsigned* err, unsigned bit) {
  if (err) __hip_atomic_fetch_or(err, bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int sanitize_parent(int pa, int k, unsigned* err) {
  if (pa >= -1 && pa < k) return pa;
  report(err, kDevErrBadTree);
  return -1;
}

struct AloneParams {
  int n_tree, vocab, max_depth;
  double temp;
  const int *tokens, *parent;
  const float *logits, *draft, *uniforms;
  const int* draft_row;  // or null: row b*n_tree + k
  long long n_draft_rows;
  double* resid;  // [batch][2][vocab] unnormalised residuals (ping-pong)
  int *out_path, *out_len, *out_bonus;
  unsigned* err;  // the workspace's sticky device error word
};

inline AloneParams alone_params(const AcceptArgs& a, double* resid) {
  AloneParams p;
  p.n_tree = a.n_tree; p.vocab = a.vocab; p.max_depth = a.max_depth;
  p.temp = (double)a.temperature;
  p.tokens = a.tokens; p.parent = a.parent;
  p.logits = a.logits; p.draft = a.draft_probs; p.uniforms = a.uniforms;
  p.draft_row = a.draft_row; p.n_draft_rows = a.n_draft_rows;
  p.resid = resid;
  p.out_path = a.out_path; p.out_len = a.out_len; p.out_bonus = a.out_bonus;
  p.err = static_cast<unsigned*>(a.workspace);
  return p;
}

template <int THREADS>
struct AloneShared {
  static_assert(THREADS >= JK_MAX_TREE, "a thread per node");
  int parent[JK_MAX_TREE];
  double red[THREADS / 64];
  double upto[THREADS];
  int found;
};

template <int THREADS>
__device__ __forceinline__ double block_sum_f64(double v, double* red) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  const int w = threadIdx.x >> 6;
  __syncthreads();  // protects red[] against the previous use
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  double r = 0.0;
  for (int i = 0; i < THREADS / 64; ++i) r += red[i];
  return r;
}
template <int THREADS>
__device__ __forceinline__ float block_max_f32(float v, double* red) {
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[w] = (double)v;
  __syncthreads();
  float r = -INFINITY;
  for (int i = 0; i < THREADS / 64; ++i) r = fmaxf(r, (float)red[i]);
  return r;
}

// row_stats(r, max, z): the largest of logits row r (of tree b) / T, 0 if there is none, and the sum of the exponentials of
// the row's distances from it; every thread calls it and gets the same.
template <int THREADS, class RowStats>
__device__ __forceinline__ void walk_alone(const AloneParams& p, int b, AloneShared<THREADS>& sh, RowStats row_stats) {
  const int tid = threadIdx.x;
  const int N = p.n_tree, V = p.vocab;
  const int rows = N + 1;
  if (tid < N) {
    sh.parent[tid] = sanitize_parent(p.parent[(long long)b * N + tid], tid, p.err);
    const int t = p.tokens[(long long)b * N + tid];
    if (t < 0 || t >= V) report(p.err, kDevErrBadToken);
  }
  __syncthreads();

  const int* tok = p.tokens + (long long)b * N;
  const float* uni = p.uniforms + (long long)b * rows;
  double* res0 = p.resid + (long long)b * 2 * V;

  int c = -1, len = 0;
  // current distribution at c: either softmax of row c+1 (fresh) or resid[cur] / res_s
  bool fresh = true;
  int cur = 0;
  double res_s = 1.0;
  double row_max = 0.0;  // max of row / T
  double row_z = 1.0;
  const float* row = nullptr;

  auto load_row_stats = [&](int r) {
    row = p.logits + ((long long)b * rows + r) * V;
    row_stats(r, row_max, row_z);
  };
  // probability of token v under the current distribution (every thread may call it)
  auto prob = [&](int v) -> double {
    if (fresh) return exp((double)row[v] / p.temp - row_max) / row_z;
    return res0[(long long)cur * V + v] / res_s;
  };

  load_row_stats(0);
  int k = 0;  // children of c are searched from k upwards (topological numbering)
  while (len < p.max_depth) {  // (at the cap the token after c comes from c's own row, untouched)
    // next child of c, left to right
    int child = -1;
    for (int j = k; j < N; ++j)
      if (sh.parent[j] == c) { child = j; break; }
    if (child < 0) break;
    const int x = min(max(tok[child], 0), V - 1);  // a token id outside the vocabulary must not fault
    long long qr = (long long)b * N + child;
    if (p.draft_row) {
      qr = p.draft_row[qr];
      qr = qr < 0 ? 0 : (qr >= p.n_draft_rows ? p.n_draft_rows - 1 : qr);
    }
    const float* qk = p.draft + qr * V;
    const double lhs = (double)uni[child] * (double)qk[x];
    const double rhs = prob(x);
    if (lhs < rhs) {
      if (tid == 0) p.out_path[(long long)b * p.max_depth + len] = child;
      ++len;
      c = child;
      k = child + 1;
      fresh = true;
      load_row_stats(c + 1);
      continue;
    }
    // rejected: r = max(0, p - q_k), written unnormalised to the other buffer
    double* dst = res0 + (long long)(fresh ? 0 : (cur ^ 1)) * V;
    double part = 0.0;
    for (int v = tid; v < V; v += THREADS) {
      const double r = fmax(0.0, prob(v) - (double)qk[v]);
      dst[v] = r;
      part += r;
    }
    const double s = block_sum_f64<THREADS>(part, sh.red);  // its barriers also order dst[] for later readers
    if (s > 0.0) {
      cur = fresh ? 0 : (cur ^ 1);
      fresh = false;
      res_s = s;
    }
    k = child + 1;
  }

  // ---- bonus token: smallest v whose cumulative probability exceeds u * total
  const int seg = (V + THREADS - 1) / THREADS;
  const int s0 = min(V, tid * seg), s1 = min(V, s0 + seg);
  double part = 0.0;
  for (int v = s0; v < s1; ++v) part += prob(v);
  sh.upto[tid] = part;
  if (tid == 0) sh.found = -1;
  __syncthreads();
  // inclusive scan over the threads' sums (Hillis-Steele in LDS)
  for (int o = 1; o < THREADS; o <<= 1) {
    const double add = (tid >= o) ? sh.upto[tid - o] : 0.0;
    __syncthreads();
    sh.upto[tid] += add;
    __syncthreads();
  }
  const double total = sh.upto[THREADS - 1];
  const double target = (double)uni[N] * total;
  const double excl = (tid == 0) ? 0.0 : sh.upto[tid - 1];
  if (s1 > s0 && excl <= target && sh.upto[tid] > target) {
    double run = excl;
    int found = -1;
    for (int v = s0; v < s1; ++v) {
      run += prob(v);
      if (run > target) { found = v; break; }
    }
    // rounding between the scanned and the re-added sums can leave the segment without a hit
    if (found < 0) found = s1 - 1;
    atomicMax(&sh.found, found);
  }
  __syncthreads();
  const int hit = sh.found;  // every thread reads the same value before anyone may change it
  __syncthreads();
  if (hit < 0) {
    // u * total not below the last cumulative value: largest v with positive probability
    int last = -1;
    for (int v = s0; v < s1; ++v)
      if (prob(v) > 0.0) last = v;
    if (last >= 0) atomicMax(&sh.found, last);
  }
  __syncthreads();
  if (tid == 0) {
    for (int i = len; i < p.max_depth; ++i) p.out_path[(long long)b * p.max_depth + i] = -1;
    p.out_len[b] = len;
    p.out_bonus[b] = sh.found < 0 ? 0 : sh.found;
  }
}

}  // namespace dev
}  // namespace jk
