// Speculative-sampling acceptance walk, cooperative version (gfx950).
//
// Same rule as the single-workgroup walk (Section 2.1 steps 2-3 of the paper:
// accept with probability min(1, p/q), continue with norm(max(0, p - q)) after
// a rejection; siblings tried left to right, Section 3.1.2), spread over W
// workgroups per tree.  A thread owns PER consecutive vocabulary entries and keeps
// their current probabilities in registers as fp64, so that a rejection only
// streams the rejected node's draft distribution from HBM.  Logits rows are read
// lazily: only the rows of nodes the walk may reach next.
//
// Every workgroup follows the same control flow.  Scalars that depend on the
// whole vocabulary (row maximum and normaliser, residual mass) are exchanged
// through a small table in the workspace: each workgroup publishes its partial
// under a tag that is unique to the call and the exchange number, then reads the
// W partials once all tags have appeared.  All workgroups reduce the same values
// in the same order, so they take identical decisions.
//
// What bounds it: the chain of exchanges, 1.5 - 2 us each through memory (a store that every
// XCD can see, then a poll that sees it), not the bytes.  So the walk makes as few as it can and
// hides its other work behind them:
//   - an exchange carries, beside what it is needed for, the statistics of the row that comes
//     next if the next candidate is accepted (worked out while the first part is on its way),
//     so that an accepted candidate behind a rejection or behind the start costs no exchange;
//   - the residual's owner of the next candidate's token publishes its value with the residual
//     mass: the test needs nothing else;
//   - the final draw takes the slices' sums from the last exchange;
//   - the draft and logits slices of the next candidate and of its first child are asked for
//     before the exchange in front of them.
// Reductions across a wave are DPP moves (a shuffle through LDS takes several times as long), one
// wave polls and reduces for the workgroup.  Measured (MI355X, us per call, twelve draws of the inputs, the same ones for
// both, repeats within 0.7 %): one 60-node tree over a 128K vocabulary 18.1 -> 15.6 in the mean (1.13 to 1.20 times as fast; a
// draw takes 11.8 to 21.7, by its number of exchanges), eight 100-node trees over a 32K vocabulary 30.9 -> 24.4 (1.14 to
// 1.35 times; 17.8 to 29.6), by asking for the words of an exchange together (a poll used to be three or four trips to memory
// in a row) and by their layout.  (Tried: a tree's
// workgroups on one XCD, exchanges through its L2: no faster than that, and one XCD's share of the memory bandwidth
// is too little for large vocabularies: one tree over 128K 25 - 31 us.)
//
// Waiting is bounded: if a partner never shows up (the W workgroups of a tree are not all
// resident) the walk gives up and reports accept_len = -1 instead of hanging; the last workgroup
// of a tree to finish finds out and moves the call number on (see TreeWords), so a call that
// gave up leaves nothing behind that a later call could mistake.
#include "jk_internal.h"
#include "jk_wave.h"

namespace jk {
namespace {

constexpr int kCoopThreads = 256;
constexpr int kCoopWaves = kCoopThreads / 64;
// Polls before giving up: 27 ms at 0.21 us each (measured behind a kernel of another stream that left 8 CUs to the walk: 4096
// polls end after 0.85 ms, 32768 after 6.9; more where the memory is busy).  Other streams' kernels hold partners up for
// milliseconds, and what gives up has no result.  To be measured again when a poll or the words' layout changes.
constexpr unsigned kDefaultSpinLimit = 1u << 17;

// The workgroups' contributions to an exchange, word by word: a wave that looks for one word of all of them reads 512
// bytes in a row (64 bytes per workgroup, all its words together, were 7 - 11 % slower).  Every 64-bit word holds the exchange's 32-bit tag
// and 32 bits of payload and is written and read with one access, so a reader that sees the tag
// also sees the payload that belongs to it: no fences and no ordering between the words are needed.
// Words 0 - 3 are what the exchange is for: a residual's mass (a double in two words) and the
// residual's value at the next candidate's token (likewise; only the owner's counts), or a logits row's sum of
// exponentials (two words) and largest logit (word 2).  Words 4 - 6: the same of the row that may come next.
struct Table {
  unsigned long long word[8][64];
};

// Per-tree words in the workspace header.  `epoch` numbers the calls: every exchange of a call is
// tagged with epoch + 1, and only the LAST workgroup of the tree to finish moves it on (it counts
// the finished ones, and those that gave up, in `finish` and returns that to zero), so that workgroups that start late -
// even after the others have given up and left - still read the call's own epoch and can never
// publish a tag that a later call would take for its own.  The length and the bonus token are written
// through to memory by the workgroups that know them; where one gave up, the last to finish overwrites them.
struct TreeWords {  // 128 bytes: a line of its own
  unsigned long long epoch;
  unsigned finish;  // finished workgroups, and << 16 those that gave up
  unsigned pad[29];
};

// What a tree owns in the workspace: its words and two exchange tables of up to 64 slots.  Tree b's
// block sits at b * sizeof(TreeBlock) whatever the batch size, mode or vocabulary of a call is, and
// the blocks of all kCoopMaxTrees trees are set aside in every acceptance workspace (see
// accept_coop_bytes), so calls of different shapes and modes can share one workspace.
struct TreeBlock {  // 8320 bytes
  TreeWords words;
  Table tables[2];
};

struct CoopParams {
  int n_tree, vocab, max_depth, W;
  double inv_temp;  // 1 / temperature
  const int *tokens, *parent;
  const float *logits, *draft, *uniforms;
  const int* draft_row;  // or null: row b*n_tree + k of draft
  long long n_draft_rows;
  TreeBlock* trees;  // [batch] words and exchange tables of each tree (zero before the first use of the workspace)
  unsigned spin_limit;
  int *out_path, *out_len, *out_bonus;
  unsigned* err;  // the workspace's sticky device error word
};

using dev::wave_max;
using dev::wave_sum;

// inclusive sums over the lanes: rows of 16 by shifts, then the rows' totals broadcast into the rows behind them
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp64_rows(double v) {  // 0 where there is no source lane
  const long long b = __double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)b, CTRL, ROWS, 0xf, false);
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWS, 0xf, false);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ double wave_scan(double v) {
  v += dpp64_rows<0x111, 0xf>(v);  // row_shr:1
  v += dpp64_rows<0x112, 0xf>(v);
  v += dpp64_rows<0x114, 0xf>(v);
  v += dpp64_rows<0x118, 0xf>(v);
  v += dpp64_rows<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
  v += dpp64_rows<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
  return v;
}
__device__ __forceinline__ double lane_before(double v) { return dpp64_rows<0x138, 0xf>(v); }  // wave_shr:1
__device__ __forceinline__ double lane_value(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)b, lane), hi = (unsigned)__builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

__device__ __forceinline__ double pair_to_double(unsigned lo, unsigned hi) {
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

template <int PER>
__global__ __launch_bounds__(kCoopThreads, 2) void walk_sample_coop_kernel(CoopParams p) {
  constexpr int SLICE = kCoopThreads * PER;
  __shared__ int par_s[JK_MAX_TREE];
  __shared__ int tok_s[JK_MAX_TREE];
  __shared__ int qrow_s[JK_MAX_TREE];
  __shared__ float uni_s[JK_MAX_TREE + 1];
  __shared__ double red_d[2][kCoopWaves];
  __shared__ float red_f[2][kCoopWaves];
  __shared__ double xs[64];    // the slices' sums under the current distribution
  // What the polling wave found.  A wave may be two finds ahead of another one (a row adopted right behind another), so
  // each kind has its own words.
  __shared__ double got_row[2][2], got_res[2];
  __shared__ int got_ok[3];
  __shared__ int s_found;
  __shared__ int s_lp[kCoopWaves];
  __shared__ double pv_s;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int W = p.W;
  const int b = blockIdx.x / W, w = blockIdx.x % W;
  const int N = p.n_tree, V = p.vocab, rows = N + 1;
  const int v0 = w * SLICE + tid * PER;  // my first vocabulary entry

  // PER consecutive floats of a row (rows are not aligned in general: loads of four at any multiple of four bytes)
  typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
  auto load_slice = [&](float (&dst)[PER], const float* row, float fill) {
    if (PER >= 4 && v0 + PER <= V) {
#pragma unroll
      for (int u = 0; u < PER; u += 4) {
        const f4 x = *reinterpret_cast<const f4*>(row + v0 + u);
#pragma unroll
        for (int i = 0; i < 4 && u + i < PER; ++i) dst[u + i] = x[i];
      }
    } else {
#pragma unroll
      for (int u = 0; u < PER; ++u) dst[u] = v0 + u < V ? row[v0 + u] : fill;
    }
  };
  auto row_of = [&](int r) { return p.logits + ((long long)b * rows + r) * V; };

  float lg[PER];
  load_slice(lg, row_of(0), -INFINITY);  // (the first row is on its way before anything else is known)
  int pa_reg = -1, tok_reg = 0;
  TreeWords* tw = &p.trees[b].words;
  const unsigned long long epoch = __hip_atomic_load(&tw->epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (tid < N) {
    pa_reg = p.parent[(long long)b * N + tid];
    tok_reg = p.tokens[(long long)b * N + tid];
    long long r = (long long)b * N + tid;
    if (p.draft_row) {
      r = p.draft_row[r];
      r = r < 0 ? 0 : (r >= p.n_draft_rows ? p.n_draft_rows - 1 : r);  // a bad row number must not fault
    }
    par_s[tid] = (pa_reg >= -1 && pa_reg < tid) ? pa_reg : -1;
    tok_s[tid] = min(max(tok_reg, 0), V - 1);  // a token id outside the vocabulary must not fault
    qrow_s[tid] = (int)r;
    if (w == 0) {  // both repairs are recorded in the workspace's error word
      if (par_s[tid] != pa_reg) __hip_atomic_fetch_or(p.err, kDevErrBadTree, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (tok_s[tid] != tok_reg) __hip_atomic_fetch_or(p.err, kDevErrBadToken, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  if (tid <= N) uni_s[tid] = p.uniforms[(long long)b * rows + tid];
  __syncthreads();
  auto q_of = [&](int k) { return p.draft + (long long)qrow_s[k] * V; };  // the draft distribution of node k

  // smallest j >= from with parent c, or -1: every wave looks at all (at most 128) nodes, two
  // per lane, so no barrier is needed and all waves get the same answer
  auto find_child = [&](int c, int from) -> int {
    const bool h0 = lane < N && lane >= from && par_s[lane] == c;
    const bool h1 = lane + 64 < N && lane + 64 >= from && par_s[lane + 64] == c;
    const unsigned long long m0 = __ballot(h0), m1 = __ballot(h1);
    return m0 ? __ffsll((long long)m0) - 1 : (m1 ? 63 + __ffsll((long long)m1) : -1);
  };

  // A candidate and what will be needed of it: its draft slice and value at its token, the logits slice of its own row
  // (the one that counts if it is accepted) and that row's value at its first child's token.
  struct Candidate {
    int k, first;  // node, its first child (or -1)
    float q[PER], lg[PER];
    float qx, row_x;
  };
  auto fetch = [&](Candidate& n, int k) {
    n.k = k;
    n.first = -1;
    if (k < 0) return;
    n.first = find_child(k, k + 1);
    const float *q = q_of(k), *row = row_of(k + 1);
    load_slice(n.q, q, 0.f);
    n.qx = q[tok_s[k]];
    load_slice(n.lg, row, -INFINITY);
    n.row_x = row[tok_s[n.first < 0 ? k : n.first]];
  };

  int flip = 0;  // alternates the LDS words of consecutive block reductions: one barrier each
  auto block_sum = [&](double v) {
    flip ^= 1;
    v = wave_sum(v);
    if (lane == 0) red_d[flip][wave] = v;
    __syncthreads();
    return (red_d[flip][0] + red_d[flip][1]) + (red_d[flip][2] + red_d[flip][3]);
  };
  auto block_max = [&](float v) {
    flip ^= 1;
    v = wave_max(v);
    if (lane == 0) red_f[flip][wave] = v;
    __syncthreads();
    return fmaxf(fmaxf(red_f[flip][0], red_f[flip][1]), fmaxf(red_f[flip][2], red_f[flip][3]));
  };

  // Tags: 22 bits of call epoch, 10 bits of exchange number (at most N + depth + 2 < 1024 per call).  The two tables take
  // turns from exchange to exchange and from call to call, and every exchange writes all its words.
  unsigned n_exch = 0, tag = 0;
  Table* tab = nullptr;
  auto open_exchange = [&] {
    ++n_exch;
    tag = (unsigned)(((epoch + 1) & 0x3FFFFFull) << 10) | (n_exch & 0x3FFu);
    tab = p.trees[b].tables + ((n_exch + (unsigned)epoch) & 1u);
  };
  auto put = [&](int word, unsigned payload) {
    __hip_atomic_store(&tab->word[word][w], ((unsigned long long)tag << 32) | payload, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  auto publish4 = [&](double a, double v) {  // words 0 - 3
    if (tid < 4) {
      const unsigned long long bits = (unsigned long long)__double_as_longlong(tid < 2 ? a : v);
      put(tid, (unsigned)(bits >> (32 * (tid & 1))));
    }
  };
  auto publish_row = [&](int at, double z, float m) {  // words at, at + 1 (z), at + 2 (m)
    if (tid < 3) {
      const unsigned long long bits = (unsigned long long)__double_as_longlong(z);
      put(at + tid, tid == 2 ? __float_as_uint(m) : (unsigned)(bits >> (32 * tid)));
    }
  };
  // wave 0: lane i waits for words [at, at + n) of workgroup i and returns their payloads
  auto await = [&](int at, int n, unsigned (&pay)[4]) -> bool {
    const bool in = lane < W;
    unsigned spins = 0;
    for (;;) {
      bool ok = true;
      unsigned long long v[4] = {};
      if (in) {  // (one condition around all loads: with one around each the compiler waits for a word before it asks for the next)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (i < n) v[i] = __hip_atomic_load(&tab->word[at + i][lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (i < n) {
            ok = ok & ((unsigned)(v[i] >> 32) == tag);
            pay[i] = (unsigned)v[i];
          }
      }
      if (__all(ok)) return true;
      if (++spins > p.spin_limit) return false;
      __builtin_amdgcn_s_sleep(1);
    }
  };

  double e[PER];               // exp(row / T - its slice's maximum) of the row that `e_m` belongs to
  float e_m = 0.f;
  double cur[PER];             // the current distribution
  double row_m = 0.0, row_inv = 1.0;  // of the current row: maximum of row / T, 1 / sum of exp(row / T - maximum)

  // slice statistics of a row: e[], e_m (largest logit of the slice) and the slice's sum
  auto slice_stats = [&](const float (&x)[PER]) -> double {
    float m = -INFINITY;
#pragma unroll
    for (int u = 0; u < PER; ++u) m = fmaxf(m, x[u]);
    e_m = block_max(m);
    const double ref = e_m == -INFINITY ? 0.0 : (double)e_m * p.inv_temp;
    double z = 0.0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      e[u] = exp((double)x[u] * p.inv_temp - ref);
      z += e[u];
    }
    return block_sum(z);
  };
  // everybody's statistics of a row -> its maximum, normaliser and slice sums; cur[] from e[]
  auto adopt_row = [&](int at) -> bool {
    if (wave == 0) {
      unsigned pay[4] = {0u, 0u, 0u, 0u};
      const bool ok = await(at, 3, pay);
      const float m_w = lane < W ? __uint_as_float(pay[2]) : -INFINITY;
      const float m = wave_max(m_w);
      const double ref = m == -INFINITY ? 0.0 : (double)m * p.inv_temp;
      const double z_w = lane < W ? pair_to_double(pay[0], pay[1]) * exp((m_w == -INFINITY ? 0.0 : (double)m_w * p.inv_temp) - ref) : 0.0;
      const double z = wave_sum(lane < W && m_w != -INFINITY ? z_w : 0.0);
      const double inv = 1.0 / z;
      xs[lane] = (m_w == -INFINITY ? 0.0 : z_w) * inv;
      if (lane == 0) {
        got_row[at == 4][0] = ref;
        got_row[at == 4][1] = inv;
        got_ok[at == 4] = ok;
      }
    }
    __syncthreads();
    row_m = got_row[at == 4][0];
    row_inv = got_row[at == 4][1];
    const double ref = e_m == -INFINITY ? 0.0 : (double)e_m * p.inv_temp;
    const double sc = exp(ref - row_m) * row_inv;
#pragma unroll
    for (int u = 0; u < PER; ++u) cur[u] = e[u] * sc;
    return got_ok[at == 4] != 0;
  };

  Candidate cand, ahead;
  fetch(cand, find_child(-1, 0));
  bool row_known;  // e[] and the open exchange's words 4 - 6 are the statistics of cand's own row
  // The statistics of candidate n's row, behind the exchange that is under way (zeros for none: the words are always written)
  auto look_ahead = [&](const Candidate& n) {
    double z = 0.0;
    if (n.k >= 0) z = slice_stats(n.lg);
    publish_row(4, z, n.k >= 0 ? e_m : 0.f);
  };

  int c = -1, len = 0;
  double px = 0.0;  // probability of cand's token under the current distribution
  bool alive;
  {
    const double z = slice_stats(lg);
    open_exchange();
    publish_row(0, z, e_m);
    if (tid == 3) put(3, 0u);
    double e0[PER];
    const float m0 = e_m;
#pragma unroll
    for (int u = 0; u < PER; ++u) e0[u] = e[u];
    const float row_x = row_of(0)[tok_s[cand.k < 0 ? 0 : cand.k]];
    look_ahead(cand);
    double e1[PER];
    const float m1 = e_m;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      e1[u] = e[u];
      e[u] = e0[u];
    }
    e_m = m0;
    alive = adopt_row(0);
#pragma unroll
    for (int u = 0; u < PER; ++u) e[u] = e1[u];
    e_m = m1;
    row_known = true;
    px = exp((double)row_x * p.inv_temp - row_m) * row_inv;
  }
  while (alive && cand.k >= 0) {
    const int k = cand.k;
    if ((double)uni_s[k] * (double)cand.qx < px) {
      // ---- accepted: the row of k becomes the current one, its first child the candidate
      if (tid == 0 && w == 0) p.out_path[(long long)b * p.max_depth + len] = k;
      ++len;
      c = k;
      const float row_x = cand.row_x;
      // at max_depth accepted nodes the walk stops: the token after c is drawn from c's own row
      const int next = len < p.max_depth ? cand.first : -1;
      if (row_known) {
        fetch(ahead, next);
        alive = adopt_row(4);
        row_known = false;
      } else {
        const double z = slice_stats(cand.lg);
        fetch(ahead, next);
        open_exchange();
        publish_row(0, z, e_m);
        if (tid == 3) put(3, 0u);
        double e0[PER];
        const float m0 = e_m;
#pragma unroll
        for (int u = 0; u < PER; ++u) e0[u] = e[u];
        look_ahead(ahead);
        double e1[PER];
        const float m1 = e_m;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
          e1[u] = e[u];
          e[u] = e0[u];
        }
        e_m = m0;
        alive = adopt_row(0);
#pragma unroll
        for (int u = 0; u < PER; ++u) e[u] = e1[u];
        e_m = m1;
        row_known = true;
      }
      px = exp((double)row_x * p.inv_temp - row_m) * row_inv;
      cand = ahead;
      continue;
    }
    // ---- rejected: the residual's mass, and its value at the next sibling's token
    fetch(ahead, find_child(c, k + 1));
    const int x = ahead.k >= 0 ? tok_s[ahead.k] : 0;
    double part = 0.0, at_x = 0.0, res[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      res[u] = v0 + u < V ? fmax(0.0, cur[u] - (double)cand.q[u]) : 0.0;
      part += res[u];
      if (v0 + u == x) at_x = res[u];
    }
    if (x >= v0 && x < v0 + PER) pv_s = at_x;  // (one thread of one workgroup; the sum's barrier orders it)
    const double s_w = block_sum(part);
    open_exchange();
    publish4(s_w, pv_s);
    look_ahead(ahead);
    row_known = true;
    if (wave == 0) {
      unsigned pay[4] = {0u, 0u, 0u, 0u};
      const bool ok = await(0, 4, pay);
      const double mine = lane < W ? pair_to_double(pay[0], pay[1]) : 0.0;
      const double s = wave_sum(mine);
      const int owner = __builtin_amdgcn_readfirstlane(x / SLICE);
      const double v = pair_to_double(__builtin_amdgcn_readlane(pay[2], owner), __builtin_amdgcn_readlane(pay[3], owner));
      if (s > 0.0) xs[lane] = mine * (1.0 / s);
      if (lane == 0) {
        got_res[0] = s;
        got_res[1] = v;
        got_ok[2] = ok;
      }
    }
    __syncthreads();
    alive = got_ok[2] != 0;
    const double s = got_res[0];
    if (s > 0.0) {
      const double inv = 1.0 / s;
#pragma unroll
      for (int u = 0; u < PER; ++u) cur[u] = res[u] * inv;
      px = got_res[1] * inv;
    } else if (alive && ahead.k >= 0) {
      // nothing left of the distribution: it stays as it was, and the next token's value under it has to be asked for
      double e1[PER];
      if (x >= v0 && x < v0 + PER) {
#pragma unroll
        for (int u = 0; u < PER; ++u)
          if (v0 + u == x) pv_s = cur[u];
      }
      __syncthreads();
      // (the row statistics ahead go along again: words 4 - 6 belong to the exchange that is open)
#pragma unroll
      for (int u = 0; u < PER; ++u) e1[u] = e[u];
      const float m1 = e_m;
      double z = 0.0;
#pragma unroll
      for (int u = 0; u < PER; ++u) z += e1[u];
      z = block_sum(z);
      open_exchange();
      publish4(0.0, pv_s);
      publish_row(4, z, m1);
      if (wave == 0) {
        unsigned pay[4] = {0u, 0u, 0u, 0u};
        const bool ok = await(0, 4, pay);
        const int owner = __builtin_amdgcn_readfirstlane(x / SLICE);
        const double v = pair_to_double(__builtin_amdgcn_readlane(pay[2], owner), __builtin_amdgcn_readlane(pay[3], owner));
        if (lane == 0) {
          got_res[1] = v;
          got_ok[2] = ok;
        }
      }
      __syncthreads();
      alive = got_ok[2] != 0;
      px = got_res[1];
    }
    cand = ahead;
  }
  // ---- final draw: smallest v whose cumulative probability exceeds u * total
  if (alive) {
    // workgroup i owns the crossing iff before(i) <= target < before(i) + its sum, with before(i) its left neighbour's
    // scanned sum: the intervals tile [0, total), rounding included, and every workgroup computes the same ones
    const double upto = wave_scan(lane < W ? xs[lane] : 0.0);
    const double before = lane_before(upto);
    const double total = lane_value(upto, 63);
    const double target = (double)uni_s[N] * total;
    const unsigned long long hit = __ballot(before <= target && upto > target);
    const int owner = hit ? __ffsll((long long)hit) - 1 : -1;
    const double owner_lo = hit ? lane_value(before, owner) : 0.0;
    if (w == owner) {
      const double local = target - owner_lo;
      double part = 0.0;
      int last_pos = -1;
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        if (v0 + u < V) {
          part += cur[u];
          if (cur[u] > 0.0) last_pos = v0 + u;
        }
      }
      // scan of the threads' sums: wave scan, then wave offsets
      const double incl = wave_scan(part), excl = lane_before(incl);
      flip ^= 1;
      if (lane == 63) red_d[flip][wave] = incl;
      int lp = last_pos;
      for (int o = 32; o > 0; o >>= 1) lp = max(lp, __shfl_xor(lp, o));
      if (lane == 0) s_lp[wave] = lp;
      if (tid == 0) s_found = -1;
      __syncthreads();
      double off = 0.0;
      for (int i = 0; i < wave; ++i) off += red_d[flip][i];
      const double lo = off + excl, hi = off + incl;
      if (lo <= local && hi > local) {
        double run = lo;
        int found = -1;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
          if (v0 + u < V) {
            run += cur[u];
            if (found < 0 && run > local) found = v0 + u;
          }
        }
        if (found < 0) found = last_pos;  // rounding between the scanned and the re-added sums
        atomicMax(&s_found, found);
      }
      __syncthreads();
      if (tid == 0) {
        // (the slice's published sum and the re-added one may differ in the last place: then its last entry with p > 0)
        const int token = s_found >= 0 ? s_found : max(max(s_lp[0], s_lp[1]), max(s_lp[2], s_lp[3]));
        __hip_atomic_store(&p.out_bonus[b], token < 0 ? 0 : token, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    if (w == 0 && tid == 0) {
      if (owner < 0) __hip_atomic_store(&p.out_bonus[b], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // no entry with p > 0
      for (int i = len; i < p.max_depth; ++i) p.out_path[(long long)b * p.max_depth + i] = -1;
      __hip_atomic_store(&p.out_len[b], len, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  // ---- the end of this workgroup: say so; where one of the tree gave up, the last to finish takes the results back
  if (tid == 0) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the results went through to memory before the count can tell anybody)
    const unsigned mine = 1u + (alive ? 0u : 0x10000u);
    const unsigned all = __hip_atomic_fetch_add(&tw->finish, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + mine;
    if ((all & 0xFFFFu) == (unsigned)W) {
      __hip_atomic_store(&tw->finish, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (all >> 16) {
        __hip_atomic_store(&p.out_len[b], -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&p.out_bonus[b], -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_or(p.err, kDevErrWalkWait, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      __hip_atomic_store(&tw->epoch, epoch + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

}  // namespace

// The blocks of kCoopMaxTrees trees are part of every acceptance workspace, whatever a call's mode and
// batch size: nothing else is ever laid over them, so greedy and sampling calls of any shapes can
// take turns on one workspace without disturbing the words the cooperative walk keeps between calls.
constexpr int kCoopMaxTrees = 512;
size_t accept_coop_bytes() { return (size_t)kCoopMaxTrees * sizeof(TreeBlock); }

bool accept_coop_plan(int batch, int vocab, int cus, int* W, int* per) {
  if (batch > kCoopMaxTrees) return false;
  int most = (2 * cus) / batch;  // two workgroups per CU are resident together
  if (most > 64) most = 64;
  // Entries per thread: fewer of them mean more workgroups to wait for, more of them longer rows of exponentials.  (us, trees x
  // entries: 8 x 32000 with 2 a thread (63 workgroups a tree) 24.4, 4 (32) 23.1; 16 x 32000 with 4 25.2, 8 27.6; 64 x 8000
  // 30.6, 34.3.)  Two only where every workgroup has a CU to itself: 1 x 8000 12.4, with four 13.3; 8 x 8000 20.4 and 22.7.
  for (int n = 2; n <= 16; n *= 2) {
    const int need = (vocab + kCoopThreads * n - 1) / (kCoopThreads * n);
    if (need <= most && (n > 2 || need * batch <= cus)) {
      *W = need;
      *per = n;
      return true;
    }
  }
  return false;
}

hipError_t launch_accept_coop(const AcceptArgs& a, void* coop_ws, int W, int per, hipStream_t stream) {
  CoopParams cp;
  cp.err = static_cast<unsigned*>(a.workspace);
  cp.n_tree = a.n_tree; cp.vocab = a.vocab; cp.max_depth = a.max_depth; cp.W = W;
  cp.inv_temp = 1.0 / (double)a.temperature;
  cp.tokens = a.tokens; cp.parent = a.parent;
  cp.logits = a.logits; cp.draft = a.draft_probs; cp.uniforms = a.uniforms;
  cp.draft_row = a.draft_row; cp.n_draft_rows = a.n_draft_rows;
  cp.trees = static_cast<TreeBlock*>(coop_ws);
  cp.spin_limit = tuning().spin_limit >= 0 ? (unsigned)tuning().spin_limit : kDefaultSpinLimit;
  cp.out_path = a.out_path; cp.out_len = a.out_len; cp.out_bonus = a.out_bonus;
  const dim3 grid((unsigned)(a.batch * W)), block(kCoopThreads);
  switch (per) {
    case 2: hipLaunchKernelGGL(walk_sample_coop_kernel<2>, grid, block, 0, stream, cp); break;
    case 4: hipLaunchKernelGGL(walk_sample_coop_kernel<4>, grid, block, 0, stream, cp); break;
    case 8: hipLaunchKernelGGL(walk_sample_coop_kernel<8>, grid, block, 0, stream, cp); break;
    case 16: hipLaunchKernelGGL(walk_sample_coop_kernel<16>, grid, block, 0, stream, cp); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Calibration: a pure 128-bit streaming read of `bytes` bytes (nothing is computed or written
// unless the data happen to hash to a magic value), the ceiling any HBM-bound kernel of the same
// size can be compared with.
typedef unsigned int probe_u32x4 __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(256) void stream_read_kernel(const probe_u32x4* __restrict__ src, size_t n_chunks,
                                                          unsigned* sink) {
  probe_u32x4 acc = {0u, 0u, 0u, 0u};
  const size_t stride = (size_t)gridDim.x * 256;
#pragma unroll 4
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n_chunks; i += stride) acc += src[i];
  if ((acc.x ^ acc.y ^ acc.z ^ acc.w) == 0x9E3779B9u) sink[0] = acc.x;
}
hipError_t launch_stream_read(const void* src, size_t bytes, void* sink, hipStream_t stream) {
  const size_t n = bytes / 16;
  if (n == 0) return hipSuccess;
  const unsigned grid = (unsigned)((n + 1023) / 1024 < 16384 ? (n + 1023) / 1024 : 16384);  // ~4 chunks per thread
  hipLaunchKernelGGL(stream_read_kernel, dim3(grid), dim3(256), 0, stream, static_cast<const probe_u32x4*>(src), n,
                     static_cast<unsigned*>(sink));
  return hipGetLastError();
}

// zero fill as a kernel (safe inside HIP-graph capture, unlike a memset node)
__global__ void zero_fill_kernel(unsigned long long* p, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0ull;
}
hipError_t launch_zero_fill(void* p, size_t bytes, hipStream_t stream) {
  const size_t n = bytes / 8;
  if (n == 0) return hipSuccess;
  const unsigned grid = (unsigned)((n + 255) / 256 < 1024 ? (n + 255) / 256 : 1024);
  hipLaunchKernelGGL(zero_fill_kernel, dim3(grid), dim3(256), 0, stream, static_cast<unsigned long long*>(p), n);
  return hipGetLastError();
}

}  // namespace jk
