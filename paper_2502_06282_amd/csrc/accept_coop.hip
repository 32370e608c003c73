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
// What bounds it: the chain of exchanges, each a trip through memory (a store that every XCD can see, then a poll that
// sees it: 0.8 us) and, with as much time again, the instructions between one and the next, which a lone wave per SIMD
// issues every five to eight cycles.  So the walk makes few exchanges and keeps long chains out of their way:
//   - an exchange carries, beside what it is needed for, the statistics of the row that comes
//     next if the next candidate is accepted (worked out while the first part is on its way),
//     so that an accepted candidate behind a rejection or behind the start costs no exchange;
//   - the residual's owner of the next candidate's token publishes its value with the residual
//     mass: the test needs nothing else;
//   - the final draw takes the slices' sums from the last exchange;
//   - references of exponentials are powers of two (see Reference): no exponential between a wait and what it waits for;
//   - nodes are looked up in a table (see Node);
//   - a thread at the end of the vocabulary reads entries that are not its own instead of none (see Part): in a branch
//     the compiler waited for every load under way, and every exchange waits for that workgroup.
// Reductions across a wave are DPP moves (a shuffle through LDS takes several times as long), one wave polls and reduces for
// the workgroup.  Measured (MI355X, us per call, the mean of six draws, before the last three of these and now; a draw takes
// 12 to 28, by its number of exchanges): one 60-node tree over a 128K vocabulary 17.6 / 15.8, eight 100-node trees over 32K
// 22.5 / 20.5, one tree over 32K 12.5 / 11.3, sixteen 27.0 / 25.1.
// What a walk starts from - words, table, the first two rows - in one trip to memory instead of three or four: 24 drawn
// calls 1.021 times as fast (0.3 - 6 %).  The first draft slice in that trip as well, and the table made beside the first
// exchange: 2 - 3 % faster with a table of rows, as much slower without.  Tried on top of it and slower: both possible next
// candidates asked for before the outcome is known, with a wave of its own that polls (a wave's loads complete in order, so
// one that has asked for a slice polls behind it): the CU's address unit takes as long for their loads as the walk then
// waits less (16.5 against 14.6); a tree's workgroups on one XCD, exchanges through its L2: one XCD's share of the memory
// bandwidth is too little for large vocabularies (one tree over 128K 25 - 31).
//
// Waiting is bounded: if a partner never shows up (the W workgroups of a tree are not all
// resident) the walk gives up and reports accept_len = -1 instead of hanging; the last workgroup
// of a tree to finish finds out and moves the call number on (see TreeWords), so a call that
// gave up leaves nothing behind that a later call could mistake.  (Many trees over large vocabularies:
// that workgroup walks the tree alone instead, see walk_sample_wide_kernel.)
#include "jk_internal.h"
#include "jk_wave.h"
#include "walk_alone.h"

namespace jk {
namespace {

constexpr int kCoopThreads = 256;
// Polls before giving up: 27 ms at 0.21 us each (measured behind a kernel of another stream that left 8 CUs to the walk: 4096
// polls end after 0.85 ms, 32768 after 6.9; more where the memory is busy).  Other streams' kernels hold partners up for
// milliseconds, and what gives up has no result.  To be measured again when a poll or the words' layout changes.
constexpr unsigned kDefaultSpinLimit = 1u << 17;
// Of walk_sample_wide_kernel, which has a result all the same: 1.7 ms, where its last workgroup takes 0.3 - 1.4 for a tree alone.
constexpr unsigned kWideSpinLimit = 1u << 13;

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

// The reference of a few logits' exponentials is a power of two near the exponential of the largest: sums with different
// references are put together by changing exponents (an exponential there is a chain of 40 dependent instructions), and
// a wave needs no other wave's maximum for its own.  exp(x / T) = 2^k exp(x / T - hi - lo).
struct Reference {
  double k, hi, lo;
};
__device__ __forceinline__ bool whole_exponent(double x) { return fabs(x) < 1099511627776.0; }
__device__ __forceinline__ double exponent_of(float m, double inv_temp) {  // of the reference for a largest logit m
  const double x = (double)m * inv_temp, k = x * 1.4426950408889634;
  // (Beyond 2^40 a whole exponent would be too far off.  Two floats that differ are at least 2^16 apart there, divided by
  // T: of sums that differ in their largest logits one is nothing beside the other.)
  return whole_exponent(x) ? rint(k) : k;
}
__device__ __forceinline__ Reference reference_of(float m, double inv_temp) {
  constexpr double kLn2 = 0.6931471805599453;
  const double x = (double)m * inv_temp;
  Reference r;
  r.k = exponent_of(m, inv_temp);
  r.hi = whole_exponent(x) ? r.k * kLn2 : (m == -INFINITY ? 0.0 : x);  // (only -inf: nothing sensible to subtract)
  r.lo = whole_exponent(x) ? fma(r.k, kLn2, -r.hi) : 0.0;
  return r;
}
__device__ __forceinline__ double exp_from(float x, double inv_temp, const Reference& r) {
  return exp(fma((double)x, inv_temp, -r.hi) - r.lo);
}
// 2^(k - K) v, K the largest k
__device__ __forceinline__ double scaled_down(double v, double k, double K) { return ldexp(v, (int)fmax(k - K, -4096.0)); }

// What a walk needs of a node.  Looked up step by step in the tree's arrays it took 0.4 us a candidate, a chain of some
// hundred instructions of a lone wave per SIMD; one wave makes the table while the first row is on its way.
struct Node {
  int next, first;      // the next of its siblings, the first of its children, or -1
  int tok, tok_first;   // its token, its first child's (its own, if it has none)
  long long draft;      // where its draft distribution begins
  int uni, pad;         // the bits of its uniform number
};
struct NodeTable {
  int4 half[2][JK_MAX_TREE + 1];     // node k's at k + 1; the root's first child at 0
  unsigned kids[JK_MAX_TREE + 1][4];  // a bit per child
};

// A workgroup of a tree's: its place, the tree, and its side of the exchanges
struct Walk {
  const CoopParams& p;
  NodeTable& table;
  const int tid, lane, wave, W, b, w, N, V;
  TreeWords* tw;
  unsigned long long epoch;
  float uni_last;
  int lane_zero = 0;
  unsigned n_exch = 0, tag = 0;
  Table* tab = nullptr;

  __device__ __forceinline__ Walk(const CoopParams& params, NodeTable& nodes, int W, int b, int w, int n_tree, int vocab)
      : p(params), table(nodes), tid(threadIdx.x), lane(tid & 63), wave(__builtin_amdgcn_readfirstlane(tid >> 6)), W(W), b(b),
        w(w), N(n_tree), V(vocab) {}
  __device__ __forceinline__ const float* row_of(int r) const { return p.logits + ((long long)b * (N + 1) + r) * V; }
  // What a walk starts from is asked for in one trip to memory: a value that the compiler knows to be the same in all lanes it
  // moves to a scalar register at once, and waits for everything asked for before it.  So these are different ones, to it,
  // until settle().
  __device__ __forceinline__ void load_words() {
    tw = &p.trees[b].words;
    asm volatile("" : "=v"(lane_zero) : "0"(0));
    epoch = __hip_atomic_load(&tw->epoch + lane_zero, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uni_last = p.uniforms[(long long)b * (N + 1) + N + lane_zero];
  }
  __device__ __forceinline__ void settle() {
    const unsigned lo = __builtin_amdgcn_readfirstlane((int)(unsigned)epoch), hi = __builtin_amdgcn_readfirstlane((int)(epoch >> 32));
    epoch = (unsigned long long)hi << 32 | lo;
    uni_last = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(uni_last)));
  }
  // What the table is made of, nodes lane and lane + 64; and, by the same wave, the table, in front of a barrier
  struct Nodes {
    int par[2], tok[2], uni[2], draft[2];
  };
  __device__ __forceinline__ void ask_nodes(Nodes& x, const int* parent, const int* tokens, const float* uniforms, const int* draft_row) const {
    const int* rows = draft_row ? draft_row : parent;  // (asked for without a branch, see load_words)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k = min(lane + 64 * h, N - 1);
      const long long at = (long long)b * N + k;
      x.par[h] = parent[at];
      x.tok[h] = tokens[at];
      x.uni[h] = __float_as_int(uniforms[at + b]);
      x.draft[h] = rows[at];
    }
  }
  template <bool EARLY = false>  // asked for in a branch of its own
  __device__ __forceinline__ void make_table(Nodes x) {
    for (int i = lane; i <= N; i += 64) *reinterpret_cast<uint4*>(table.kids[i]) = make_uint4(0u, 0u, 0u, 0u);
    auto in_order = [] { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); };  // (LDS operations of a wave complete in order)
    in_order();
    int par[2], tok[2], uni[2];
    long long draft[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (EARLY) asm volatile("" : "+v"(x.par[h]), "+v"(x.tok[h]), "+v"(x.uni[h]), "+v"(x.draft[h]));  // (else widened, and waited for, where it was asked for)
      par[h] = x.par[h];
      tok[h] = x.tok[h];
      uni[h] = x.uni[h];
      draft[h] = x.draft[h];
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k = lane + 64 * h, pa = par[h], tk = tok[h];
      par[h] = (pa >= -1 && pa < k) ? pa : -1;
      tok[h] = min(max(tk, 0), V - 1);  // a token id outside the vocabulary must not fault
      if (p.draft_row) draft[h] = draft[h] < 0 ? 0 : (draft[h] >= p.n_draft_rows ? p.n_draft_rows - 1 : draft[h]);  // nor a bad row
      else draft[h] = (long long)b * N + k;
      if (k >= N) continue;
      if (w == 0) {  // both repairs are recorded in the workspace's error word
        if (par[h] != pa) __hip_atomic_fetch_or(p.err, kDevErrBadTree, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (tok[h] != tk) __hip_atomic_fetch_or(p.err, kDevErrBadToken, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      atomicOr(&table.kids[par[h] + 1][k >> 5], 1u << (k & 31));
      table.half[0][k + 1].z = tok[h];
    }
    in_order();
    auto lowest = [](const uint4& m, int above) {  // the lowest bit set beyond `above`
      const unsigned words[4] = {m.x, m.y, m.z, m.w};
      int at = -1;
#pragma unroll
      for (int i = 3; i >= 0; --i) {
        const unsigned beyond = above < 32 * i ? ~0u : (above >= 32 * i + 31 ? 0u : ~0u << (above - 32 * i + 1));
        const unsigned bits = words[i] & beyond;
        at = bits ? 32 * i + __ffs((int)bits) - 1 : at;
      }
      return at;
    };
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k = lane + 64 * h;
      if (k >= N) continue;
      const int next = lowest(*reinterpret_cast<const uint4*>(table.kids[par[h] + 1]), k);
      const int first = lowest(*reinterpret_cast<const uint4*>(table.kids[k + 1]), -1);
      const int tok_first = table.half[0][(first < 0 ? k : first) + 1].z;
      table.half[0][k + 1] = make_int4(next, first, tok[h], tok_first);
      const long long at = draft[h] * V;
      table.half[1][k + 1] = make_int4((int)at, (int)(at >> 32), uni[h], 0);
    }
    if (lane == 0) table.half[0][0].y = lowest(*reinterpret_cast<const uint4*>(table.kids[0]), -1);
  }
  __device__ __forceinline__ int first_of_root() const { return __builtin_amdgcn_readfirstlane(table.half[0][0].y); }
  __device__ __forceinline__ Node node(int k) const {
    const int4 a = table.half[0][k + 1], c = table.half[1][k + 1];
    Node n;
    n.next = __builtin_amdgcn_readfirstlane(a.x);
    n.first = __builtin_amdgcn_readfirstlane(a.y);
    n.tok = __builtin_amdgcn_readfirstlane(a.z);
    n.tok_first = __builtin_amdgcn_readfirstlane(a.w);
    n.draft = (long long)((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane(c.y) << 32 | (unsigned)__builtin_amdgcn_readfirstlane(c.x));
    n.uni = __builtin_amdgcn_readfirstlane(c.z);
    return n;
  }

  // Tags: 22 bits of call epoch, 10 bits of exchange number (at most N + depth + 2 < 1024 per call).  The two tables take
  // turns from exchange to exchange and from call to call, and every exchange writes all words that are read in it.
  __device__ __forceinline__ void open_exchange() {
    ++n_exch;
    tag = (unsigned)(((epoch + 1) & 0x3FFFFFull) << 10) | (n_exch & 0x3FFu);
    tab = p.trees[b].tables + ((n_exch + (unsigned)epoch) & 1u);
  }
  __device__ __forceinline__ void put(int word, unsigned payload) {
    __hip_atomic_store(&tab->word[word][w], ((unsigned long long)tag << 32) | payload, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ void publish4(double a, double v) {  // words 0 - 3
    if (tid < 4) {
      const unsigned long long bits = (unsigned long long)__double_as_longlong(tid < 2 ? a : v);
      put(tid, (unsigned)(bits >> (32 * (tid & 1))));
    }
  }
  struct Stats {  // of a row's slice, in the first wave: its largest logit, and the sum of its exponentials by that one's reference
    double z;
    float m;
  };
  __device__ __forceinline__ void publish_row(int at, const Stats& st) {  // words at, at + 1 (z), at + 2 (m)
    if (tid < 3) {
      const unsigned long long bits = (unsigned long long)__double_as_longlong(st.z);
      put(at + tid, tid == 2 ? __float_as_uint(st.m) : (unsigned)(bits >> (32 * tid)));
    }
  }
  // one wave: lane i waits for words [at, at + n) of workgroup i and returns their payloads
  __device__ __forceinline__ bool await(int at, int n, unsigned (&pay)[4]) const {
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
  }
  // one wave, what it awaited of a residual (words 0 - 3): its mass, its value in workgroup `owner`, and this lane's slice's part
  __device__ __forceinline__ double mass_total(const unsigned (&pay)[4], int owner, double& s, double& at_owner) const {
    const double own = lane < W ? pair_to_double(pay[0], pay[1]) : 0.0;
    s = wave_sum(own);
    const int from = __builtin_amdgcn_readfirstlane(owner);
    at_owner = pair_to_double(__builtin_amdgcn_readlane(pay[2], from), __builtin_amdgcn_readlane(pay[3], from));
    return own;
  }
  // one wave, what it awaited of a row (words 0 - 2 of `pay`): the exponent of the row's reference, its normaliser, and this
  // lane's slice's sum
  __device__ __forceinline__ void row_total(const unsigned (&pay)[4], double& K, double& z, double& mine) const {
    const float m_w = lane < W ? __uint_as_float(pay[2]) : -INFINITY;
    K = exponent_of(wave_max(m_w), p.inv_temp);
    mine = m_w == -INFINITY ? 0.0 : scaled_down(pair_to_double(pay[0], pay[1]), exponent_of(m_w, p.inv_temp), K);
    z = wave_sum(mine);
  }
  // The waves' parts put together, lane i holding part i mod WAVES (a row of 16 lanes at most: four moves)
  template <int WAVES>
  __device__ __forceinline__ static double sum_of(double v) {
    v += dev::dpp64<0xB1>(v);  // quad_perm [1,0,3,2]
    v += dev::dpp64<0x4E>(v);  // quad_perm [2,3,0,1]
    if (WAVES > 4) v += dev::dpp64<0x141>(v);  // row_half_mirror
    if (WAVES > 8) v += dev::dpp64<0x140>(v);  // row_mirror
    return v;
  }
  template <int WAVES>
  __device__ __forceinline__ Stats put_together(double z, float m) const {
    auto most = [](float v, int x) { return fmaxf(v, __int_as_float(x)); };
    Stats st;
    st.m = most(m, dev::dpp<0xB1>(__float_as_int(m)));
    st.m = most(st.m, dev::dpp<0x4E>(__float_as_int(st.m)));
    if (WAVES > 4) st.m = most(st.m, dev::dpp<0x141>(__float_as_int(st.m)));
    if (WAVES > 8) st.m = most(st.m, dev::dpp<0x140>(__float_as_int(st.m)));
    st.z = sum_of<WAVES>(scaled_down(z, exponent_of(m, p.inv_temp), exponent_of(st.m, p.inv_temp)));
    return st;
  }
  // A thread's PER consecutive vocabulary entries from v0 on: entry u is at + u, and counts from u = skip on.  (No thread
  // looks past the end of a row: those at the end read its last PER entries.  No branch, in which the compiler would wait
  // for everything under way: every exchange waits for the workgroup at the end.)
  template <int PER>
  struct Part {
    int v0, at, skip;
    __device__ __forceinline__ Part(int first, int V) : v0(first), at(min(first, V - PER)), skip(first - at) {}
    // (worked out where it is used: kept, the masks of all entries fill the scalar registers)
    __device__ __forceinline__ int first_that_counts() const {
      int s = skip;
      asm volatile("" : "+v"(s));
      return s;
    }
    __device__ __forceinline__ bool has(int x) const { return x >= v0 && x < v0 + PER; }
    // (rows are not aligned in general: loads of four at any multiple of four bytes)
    __device__ __forceinline__ void load(float (&dst)[PER], const float* row) const {
      if constexpr (PER >= 4) {
        typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll
        for (int u = 0; u < PER; u += 4) {
          const f4 x = *reinterpret_cast<const f4*>(row + at + u);
#pragma unroll
          for (int i = 0; i < 4; ++i) dst[u + i] = x[i];
        }
      } else {
#pragma unroll
        for (int u = 0; u < PER; ++u) dst[u] = row[at + u];
      }
    }
  };

  // (through to memory, like all results: a last workgroup on another XCD may have to write them anew)
  __device__ __forceinline__ void put_path(int i, int node) {
    __hip_atomic_store(&p.out_path[(long long)b * p.max_depth + i], node, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }

  // Final draw: smallest v whose cumulative probability exceeds u * total.  x: the sum of lane's slice under the current
  // distribution; cur: this thread's part of that.
  template <int PER, int WAVES>
  __device__ __forceinline__ void draw(double x, const double (&cur)[PER], const Part<PER>& mine, int len) {
    __shared__ double sum_s[WAVES];
    __shared__ int last_s[WAVES], found_s;
    // workgroup i owns the crossing iff before(i) <= target < before(i) + its sum, with before(i) its left neighbour's
    // scanned sum: the intervals tile [0, total), rounding included, and every workgroup computes the same ones
    const double upto = wave_scan(lane < W ? x : 0.0);
    const double before = lane_before(upto);
    const double total = lane_value(upto, 63);
    const double target = (double)uni_last * total;
    const unsigned long long hit = __ballot(before <= target && upto > target);
    const int owner = hit ? __ffsll((long long)hit) - 1 : -1;
    const double owner_lo = hit ? lane_value(before, owner) : 0.0;
    if (w == owner) {
      const double local = target - owner_lo;
      double part = 0.0;
      int last_pos = -1;
      const int skip = mine.first_that_counts();
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        if (u >= skip) {
          part += cur[u];
          if (cur[u] > 0.0) last_pos = mine.at + u;
        }
      }
      // scan of the threads' sums: wave scan, then wave offsets
      const double incl = wave_scan(part), excl = lane_before(incl);
      int lp = last_pos;
      for (int o = 32; o > 0; o >>= 1) lp = max(lp, __shfl_xor(lp, o));
      if (lane == 63) sum_s[wave] = incl;
      if (lane == 0) last_s[wave] = lp;
      if (tid == 0) found_s = -1;
      __syncthreads();
      double off = 0.0;
      for (int i = 0; i < wave; ++i) off += sum_s[i];
      const double lo = off + excl, hi = off + incl;
      if (lo <= local && hi > local) {
        double run = lo;
        int found = -1;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
          if (u >= skip) {
            run += cur[u];
            if (found < 0 && run > local) found = mine.at + u;
          }
        }
        if (found < 0) found = last_pos;  // rounding between the scanned and the re-added sums
        atomicMax(&found_s, found);
      }
      __syncthreads();
      if (tid == 0) {
        // (the slice's published sum and the re-added one may differ in the last place: then its last entry with p > 0)
        int token = found_s;
        if (token < 0)
          for (int i = 0; i < WAVES; ++i) token = max(token, last_s[i]);
        __hip_atomic_store(&p.out_bonus[b], token < 0 ? 0 : token, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    if (w == 0 && tid == 0) {
      if (owner < 0) __hip_atomic_store(&p.out_bonus[b], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // no entry with p > 0
      for (int i = len; i < p.max_depth; ++i) put_path(i, -1);
      __hip_atomic_store(&p.out_len[b], len, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  // The end of this workgroup, by its first thread: it says so.  True for the last one of a tree where one gave up, which takes
  // the results back
  __device__ __forceinline__ bool finish(bool alive) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the results went through to memory before the count can tell anybody)
    const unsigned mine = 1u + (alive ? 0u : 0x10000u);
    const unsigned all = __hip_atomic_fetch_add(&tw->finish, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + mine;
    if ((all & 0xFFFFu) != (unsigned)W) return false;
    __hip_atomic_store(&tw->finish, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&tw->epoch, epoch + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return all >> 16 != 0u;
  }
  __device__ __forceinline__ unsigned finished() const { return __hip_atomic_load(&tw->finish + lane_zero, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
};

// `start`: asks for the slices of rows 0 and 1, and for what a walk starts from, and makes the table
template <int PER, int THREADS, class Start>
__device__ __forceinline__ void walk_together(Walk& wk, const Start& start) {
  constexpr int SLICE = THREADS * PER, WAVES = THREADS / 64;
  __shared__ double red_d[2][WAVES];
  __shared__ float red_f[2][WAVES];
  __shared__ double xs[64];  // the slices' sums under the current distribution, still to be multiplied by xs_mul
  // What the polling wave found.  A wave may be two finds ahead of another one (a row adopted right behind another), so
  // each kind has its own words.
  __shared__ double got_row[2][2], got_res[2];
  __shared__ int got_ok[3];
  __shared__ double pv_s;

  const CoopParams& p = wk.p;
  const int tid = wk.tid, lane = wk.lane, wave = wk.wave, W = wk.W;
  const Walk::Part<PER> mine(wk.w * SLICE + tid * PER, wk.V);

  // A candidate and what will be needed of it: its draft slice and value at its token, the logits slice of its own row
  // (the one that counts if it is accepted) and that row's value at its first child's token.
  struct Candidate {
    int k;
    Node node;
    float q[PER], lg[PER];
    float qx, row_x;
  };
  // (The root's first child is node 0, since a parent comes before its children: its own row is row 1.)
  Candidate then;
  float lg[PER];
  start(mine, lg, then.lg);
  wk.settle();
  __syncthreads();
  then.k = 0;
  then.node = wk.node(0);
  mine.load(then.q, p.draft + then.node.draft);
  then.qx = p.draft[then.node.draft + then.node.tok];
  then.row_x = wk.row_of(1)[then.node.tok_first];

  auto fetch = [&](Candidate& n, int k) {
    n.k = k;
    if (k < 0) return;
    n.node = wk.node(k);
    const float *q = p.draft + n.node.draft, *row = wk.row_of(k + 1);
    mine.load(n.q, q);
    n.qx = q[n.node.tok];
    mine.load(n.lg, row);
    n.row_x = row[n.node.tok_first];
  };

  using Stats = Walk::Stats;
  struct Exponentials {  // of this thread's part of a row: 2^k e[]
    double e[PER], k;
  };
  double cur[PER];      // the current distribution
  double xs_mul = 1.0;  // (a division that only the final draw needs stays out of the polling wave's way)
  double px = 0.0;      // probability of cand's token under the current distribution
  bool alive = true;
  int flip = 0;  // alternates the LDS words of consecutive block reductions: one barrier each

  auto slice_stats = [&](const float (&x)[PER], Exponentials& out) -> Stats {
    flip ^= 1;
    float m = -INFINITY, y[PER];
    const int skip = mine.first_that_counts();
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      y[u] = u >= skip ? x[u] : -INFINITY;
      m = fmaxf(m, y[u]);
    }
    m = wave_max(m);
    const Reference ref = reference_of(m, p.inv_temp);
    out.k = ref.k;
    double z = 0.0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      out.e[u] = exp_from(y[u], p.inv_temp, ref);
      z += out.e[u];
    }
    z = wave_sum(z);
    if (lane == 0) {
      red_d[flip][wave] = z;
      red_f[flip][wave] = m;
    }
    __syncthreads();
    Stats st = {0.0, 0.f};
    if (wave == 0) st = wk.put_together<WAVES>(red_d[flip][lane % WAVES], red_f[flip][lane % WAVES]);
    return st;
  };
  // everybody's statistics of a row -> its reference, normaliser and slice sums; cur[] from the row's exponentials, and the
  // probability of the token that has this logit (its exponential is taken in front of the wait, by a reference of its own:
  // every workgroup must get the same bits)
  auto adopt_row = [&](int at, const Exponentials& ex, float logit) {
    const int kind = at == 4;
    const Reference ref = reference_of(logit, p.inv_temp);
    const double e_x = exp_from(logit, p.inv_temp, ref);
    if (wave == 0) {
      unsigned pay[4] = {0u, 0u, 0u, 0u};
      const bool ok = wk.await(at, 3, pay);
      double K, z, own;
      wk.row_total(pay, K, z, own);
      xs[lane] = own;
      if (lane == 0) {
        got_row[kind][0] = K;
        got_row[kind][1] = z;
        got_ok[kind] = ok;
      }
    }
    __syncthreads();
    const double row_k = got_row[kind][0], row_inv = 1.0 / got_row[kind][1];
    alive = got_ok[kind] != 0;
    xs_mul = row_inv;
    px = scaled_down(e_x, ref.k, row_k) * row_inv;
    const double sc = scaled_down(row_inv, ex.k, row_k);
#pragma unroll
    for (int u = 0; u < PER; ++u) cur[u] = ex.e[u] * sc;
  };

  Candidate cand;  // (`then`: fetched when the outcome names it, the next sibling or the first child)
  Exponentials ahead;    // of cand's own row, where it is known
  Stats ahead_stats = {0.0, 0.f};
  bool row_known = false;  // `ahead` and the open exchange's words 4 - 6 are those of cand's own row
  // The statistics of cand's row, behind the exchange that is under way (zeros for none: the words are always written)
  auto look_ahead = [&]() {
    ahead_stats = Stats{0.0, 0.f};
    if (cand.k >= 0) ahead_stats = slice_stats(cand.lg, ahead);
    wk.publish_row(4, ahead_stats);
    row_known = true;
  };
  // The row that becomes the current one, of which nothing is known yet, in an exchange that also carries the statistics of
  // the row of the candidate behind it
  auto exchange_row = [&](const float (&x)[PER], float row_x, const Candidate& next) {
    Exponentials now;
    const Stats st = slice_stats(x, now);
    wk.open_exchange();
    wk.publish_row(0, st);
    if (tid == 3) wk.put(3, 0u);
    cand = next;
    look_ahead();
    adopt_row(0, now, row_x);
  };

  int len = 0;
  exchange_row(lg, wk.row_of(0)[then.node.tok], then);
  while (alive && cand.k >= 0) {
    if ((double)__int_as_float(cand.node.uni) * (double)cand.qx < px) {
      // ---- accepted: its row becomes the current one, its first child the candidate
      if (tid == 0 && wk.w == 0) p.out_path[(long long)wk.b * p.max_depth + len] = cand.k;
      ++len;
      // (at max_depth accepted nodes the walk stops: the token after the last one is drawn from that one's own row)
      fetch(then, len < p.max_depth ? cand.node.first : -1);
      const float row_x = cand.row_x;
      if (row_known) {
        cand = then;
        row_known = false;
        adopt_row(4, ahead, row_x);
      } else {
#pragma unroll
        for (int u = 0; u < PER; ++u) lg[u] = cand.lg[u];
        exchange_row(lg, row_x, then);
      }
      continue;
    }
    // ---- rejected: the residual's mass, and its value at the next sibling's token
    fetch(then, cand.node.next);
    const int x = then.k >= 0 ? then.node.tok : 0;
    double part = 0.0, at_x = 0.0, res[PER];
    const int skip = mine.first_that_counts();
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      res[u] = u >= skip ? fmax(0.0, cur[u] - (double)cand.q[u]) : 0.0;
      part += res[u];
      if (mine.at + u == x) at_x = res[u];
    }
    if (mine.has(x)) pv_s = at_x;  // (one thread of one workgroup; the sum's barrier orders it)
    part = wave_sum(part);
    flip ^= 1;
    if (lane == 0) red_d[flip][wave] = part;
    __syncthreads();
    wk.open_exchange();
    if (wave == 0) wk.publish4(Walk::sum_of<WAVES>(red_d[flip][lane % WAVES]), pv_s);
    cand = then;
    look_ahead();
    if (wave == 0) {
      unsigned pay[4] = {0u, 0u, 0u, 0u};
      const bool ok = wk.await(0, 4, pay);
      double s, at_owner;
      const double own = wk.mass_total(pay, x / SLICE, s, at_owner);
      if (s > 0.0) xs[lane] = own;
      if (lane == 0) {
        got_res[0] = s;
        got_res[1] = at_owner;
        got_ok[2] = ok;
      }
    }
    __syncthreads();
    alive = got_ok[2] != 0;
    const double s = got_res[0];
    if (s > 0.0) {
      const double inv = xs_mul = 1.0 / s;
      px = got_res[1] * inv;
#pragma unroll
      for (int u = 0; u < PER; ++u) cur[u] = res[u] * inv;
    } else if (alive && cand.k >= 0) {
      // nothing left of the distribution: it stays as it was, and the next token's value under it has to be asked for
      if (mine.has(x)) {
#pragma unroll
        for (int u = 0; u < PER; ++u)
          if (mine.at + u == x) pv_s = cur[u];
      }
      __syncthreads();
      wk.open_exchange();
      wk.publish4(0.0, pv_s);
      wk.publish_row(4, ahead_stats);  // (again: words 4 - 6 belong to the exchange that is open)
      if (wave == 0) {
        unsigned pay[4] = {0u, 0u, 0u, 0u};
        const bool ok = wk.await(0, 4, pay);
        double none, at_owner;
        wk.mass_total(pay, x / SLICE, none, at_owner);
        if (lane == 0) {
          got_res[1] = at_owner;
          got_ok[2] = ok;
        }
      }
      __syncthreads();
      alive = got_ok[2] != 0;
      px = got_res[1];
    }
  }
  if (alive) wk.draw<PER, WAVES>(xs[lane] * xs_mul, cur, mine, len);
  if (tid == 0 && wk.finish(alive)) {
    __hip_atomic_store(&p.out_len[wk.b], -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&p.out_bonus[wk.b], -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_or(p.err, kDevErrWalkWait, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// The first rows are on their way before anything else is known, and the nodes: their addresses are made of the leading arguments,
// which are in scalar registers when a wave starts (a compiler option for this file, fourteen words at most).  The others take
// 0.3 us to come from memory, and which tree this is was a division.  (us, before / so: one tree of 60 nodes, 128256 entries 13.59 /
// 13.39, eight of 100, 32000 entries 21.44 / 21.21.)
template <int PER, int THREADS>
__global__ __launch_bounds__(THREADS, 2) void walk_sample_coop_kernel(const float* logits, const int* parent, const int* tokens,
                                                                      const float* uniforms, const int* draft_row, int n_tree, int vocab, int W,
                                                                      unsigned mg_w, CoopParams params) {
  __shared__ NodeTable nodes;
  const int b = mg_w ? (int)__umulhi(blockIdx.x, mg_w) : (int)blockIdx.x;
  Walk wk(params, nodes, W, b, (int)blockIdx.x - b * W, n_tree, vocab);
  walk_together<PER, THREADS>(wk, [&](const Walk::Part<PER>& mine, float (&row0)[PER], float (&row1)[PER]) __attribute__((always_inline)) {
    Walk::Nodes first_nodes;
    const float* row = logits + (long long)wk.b * (n_tree + 1) * vocab;
    mine.load(row0, row);
    mine.load(row1, row + vocab);
    if (wk.wave == 0) wk.ask_nodes(first_nodes, parent, tokens, uniforms, draft_row);
    __builtin_amdgcn_sched_barrier(0);
    wk.load_words();
    if (wk.wave == 0) wk.make_table<true>(first_nodes);
  });
}
// Eight and sixteen entries a thread, where scalar registers are short: a place in the tree made by the compiler's remainder, and
// arguments read where they are needed.  Made of b * W, b and W stay alive through the walk, and 61 and 72 scalar registers are
// spilled instead of 45 and 63.  (us, so / by leading arguments and b * W, of one card: 10 trees of 25 nodes, 128512 entries 27.08 /
// 27.41, 16 trees, 100000 entries 32.5 / 33.1.)
template <int PER, int THREADS>
__global__ __launch_bounds__(THREADS, 2) void walk_sample_long_kernel(CoopParams params) {
  __shared__ NodeTable nodes;
  Walk wk(params, nodes, params.W, (int)(blockIdx.x / (unsigned)params.W), (int)(blockIdx.x % (unsigned)params.W), params.n_tree, params.vocab);
  walk_together<PER, THREADS>(wk, [&](const Walk::Part<PER>& mine, float (&row0)[PER], float (&row1)[PER]) __attribute__((always_inline)) {
    mine.load(row0, wk.row_of(0));
    mine.load(row1, wk.row_of(1));
    wk.load_words();
    if (wk.wave == 0) {
      Walk::Nodes first_nodes;
      wk.ask_nodes(first_nodes, params.parent, params.tokens, params.uniforms, params.draft_row);
      wk.make_table(first_nodes);
    }
  });
}

// The walk of many trees over large vocabularies, where slices of 4096 entries would be more workgroups than are resident
// together: 512 threads, a workgroup for each CU at most, a slice of 8192 to 20480 entries each.  (The workgroups of a tree
// follow each other in the grid: of a call that gets only some of the CUs at most one tree waits for others to end.)  A thread
// holds the current distribution and one slice, of the candidate's draft or of the row that it brings, and looks at nothing
// ahead.  Where a workgroup gives up (another stream's kernel has its partners' CUs), those of its tree that start later do not
// wait any more, and the last one walks the tree alone, with the residuals in the workspace, as a kernel of a workgroup per tree
// would: no result is missing.  (All trees like that: 16 x 138253 1240 us, 128 x 32000 349.  The possibility costs 0 - 2 %.)
// What bounds it is the exponentials of a row (some 40 instructions of 4 cycles each) and the slices' bytes.
// Measured (us; by a workgroup per tree, in front of it a pass over all logits / like this), trees x entries: 16 x 138253
// 519 / 42, 21 x 103226 304 / 31, 32 x 128256 534 / 56, 64 x 70000 297 / 47, 128 x 32000 141 / 47, 200 x 9000 57 / 32, 250 x 12289
// 73 / 37.
constexpr int kWideThreads = 512;

template <int PER>
__global__ __launch_bounds__(kWideThreads) void walk_sample_wide_kernel(CoopParams params, dev::AloneParams) {
  constexpr int SLICE = kWideThreads * PER, WAVES = kWideThreads / 64;
  __shared__ NodeTable nodes;
  __shared__ double red_d[2][WAVES];
  __shared__ float red_f[WAVES];
  __shared__ double xs[64];  // (as above)
  __shared__ double got[2];
  __shared__ int got_ok;
  __shared__ double pv_s;

  Walk wk(params, nodes, params.W, (int)(blockIdx.x / (unsigned)params.W), (int)(blockIdx.x % (unsigned)params.W), params.n_tree, params.vocab);
  const CoopParams& p = wk.p;
  const int tid = wk.tid, lane = wk.lane, wave = wk.wave;
  const Walk::Part<PER> mine(wk.w * SLICE + tid * PER, wk.V);
  float x[PER];     // a slice
  double cur[PER];  // the current distribution
  mine.load(x, wk.row_of(0));
  wk.load_words();
  const unsigned before = wk.finished();
  if (wave == 0) {
    Walk::Nodes first_nodes;
    wk.ask_nodes(first_nodes, p.parent, p.tokens, p.uniforms, p.draft_row);
    wk.make_table(first_nodes);
    if (lane == 0) got_ok = before >> 16 == 0u;  // (where somebody of the tree has given up there is nothing to wait for)
  }
  wk.settle();
  __syncthreads();

  double xs_mul = 1.0, px = 0.0;
  bool alive = got_ok != 0;
  int flip = 0, len = 0, k = wk.first_of_root();
  Node node = wk.node(k);
  float qx = 0.f;
  // row `r`, whose slice is in x[] or on its way there, becomes the current one; behind it the draft slice of candidate k
  auto adopt_row = [&](int r) {
    const float logit = k >= 0 ? wk.row_of(r)[node.tok] : 0.f;
    float m = -INFINITY;
    const int skip = mine.first_that_counts();
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      x[u] = u >= skip ? x[u] : -INFINITY;
      m = fmaxf(m, x[u]);
    }
    m = wave_max(m);
    const Reference ref = reference_of(m, p.inv_temp);
    double z = 0.0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      cur[u] = exp_from(x[u], p.inv_temp, ref);
      z += cur[u];
      __builtin_amdgcn_sched_barrier(0);  // (one after the other: there are no registers for several at a time)
    }
    z = wave_sum(z);
    flip ^= 1;
    if (lane == 0) {
      red_d[flip][wave] = z;
      red_f[wave] = m;
    }
    __syncthreads();
    wk.open_exchange();
    if (wave == 0) wk.publish_row(0, wk.put_together<WAVES>(red_d[flip][lane % WAVES], red_f[lane % WAVES]));
    if (k >= 0) qx = (p.draft + node.draft)[node.tok];
    const Reference ref_x = reference_of(logit, p.inv_temp);
    const double e_x = exp_from(logit, p.inv_temp, ref_x);
    if (wave == 0) {
      unsigned pay[4] = {0u, 0u, 0u, 0u};
      const bool ok = wk.await(0, 3, pay);
      double K, total, own;
      wk.row_total(pay, K, total, own);
      xs[lane] = own;
      if (lane == 0) {
        got[0] = K;
        got[1] = total;
        got_ok = ok;
      }
    }
    if (k >= 0) mine.load(x, p.draft + node.draft);
    __syncthreads();
    const double row_k = got[0], row_inv = 1.0 / got[1];
    alive = got_ok != 0;
    xs_mul = row_inv;
    px = scaled_down(e_x, ref_x.k, row_k) * row_inv;
    const double sc = scaled_down(row_inv, ref.k, row_k);
#pragma unroll
    for (int u = 0; u < PER; ++u) cur[u] *= sc;
  };
  if (alive) adopt_row(0);
  while (alive && k >= 0) {
    if ((double)__int_as_float(node.uni) * (double)qx < px) {
      // ---- accepted: its row becomes the current one, its first child the candidate
      if (tid == 0 && wk.w == 0) wk.put_path(len, k);
      ++len;
      const int row = k + 1;
      mine.load(x, wk.row_of(row));
      k = len < p.max_depth ? node.first : -1;
      if (k >= 0) node = wk.node(k);
      adopt_row(row);
      continue;
    }
    // ---- rejected: the residual's mass, and its value at the next sibling's token
    k = node.next;
    if (k >= 0) node = wk.node(k);
    const int next_tok = k >= 0 ? node.tok : 0;
    double part = 0.0, at_x = 0.0, was_x = 0.0;
    const int skip = mine.first_that_counts();
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const double res = u >= skip ? fmax(0.0, cur[u] - (double)x[u]) : 0.0;
      part += res;
      if (mine.at + u == next_tok) {
        at_x = res;
        was_x = cur[u];
      }
    }
    if (mine.has(next_tok)) pv_s = at_x;  // (one thread of one workgroup; the sum's barrier orders it)
    part = wave_sum(part);
    flip ^= 1;
    if (lane == 0) red_d[flip][wave] = part;
    __syncthreads();
    auto exchange = [&](double mass) {
      wk.open_exchange();
      if (wave == 0) {
        wk.publish4(mass, pv_s);
        unsigned pay[4] = {0u, 0u, 0u, 0u};
        const bool ok = wk.await(0, 4, pay);
        double s, at_owner;
        const double own = wk.mass_total(pay, next_tok / SLICE, s, at_owner);
        if (s > 0.0) xs[lane] = own;
        if (lane == 0) {
          got[0] = s;
          got[1] = at_owner;
          got_ok = ok;
        }
      }
      __syncthreads();
      alive = got_ok != 0;
    };
    exchange(wave == 0 ? Walk::sum_of<WAVES>(red_d[flip][lane % WAVES]) : 0.0);
    const double s = got[0];
    if (s > 0.0) {
      const double inv = xs_mul = 1.0 / s;
      px = got[1] * inv;
      const int skip = mine.first_that_counts();
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        asm volatile("" : "+v"(x[u]));  // (worked out again: held since the sum, it would take as many registers as cur[])
        cur[u] = u >= skip ? fmax(0.0, cur[u] - (double)x[u]) * inv : 0.0;
      }
    } else if (alive && k >= 0) {
      // nothing left of the distribution: it stays as it was, and the next token's value under it has to be asked for
      if (mine.has(next_tok)) pv_s = was_x;
      __syncthreads();
      exchange(0.0);
      px = got[1];
    }
    if (k >= 0) {
      qx = (p.draft + node.draft)[node.tok];
      mine.load(x, p.draft + node.draft);
    }
  }
  if (alive) wk.draw<PER, WAVES>(xs[lane] * xs_mul, cur, mine, len);

  __shared__ dev::AloneShared<kWideThreads> sh;
  if (tid == 0) sh.found = wk.finish(alive);
  __syncthreads();
  if (__builtin_amdgcn_readfirstlane(sh.found) == 0) return;
  __syncthreads();
  // (fetched from the kernel's arguments here: held in scalar registers across the walk, which has none to spare, they cost
  // every call some of them)
  struct Arguments {
    CoopParams params;
    dev::AloneParams alone;
  };
  typedef __attribute__((address_space(4))) const Arguments KArgs;
  KArgs* late = (KArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(late));
  dev::AloneParams alone;
  alone.n_tree = late->alone.n_tree; alone.vocab = late->alone.vocab; alone.max_depth = late->alone.max_depth;
  alone.temp = late->alone.temp;
  alone.tokens = late->alone.tokens; alone.parent = late->alone.parent;
  alone.logits = late->alone.logits; alone.draft = late->alone.draft; alone.uniforms = late->alone.uniforms;
  alone.draft_row = late->alone.draft_row; alone.n_draft_rows = late->alone.n_draft_rows;
  alone.resid = late->alone.resid;
  alone.out_path = late->alone.out_path; alone.out_len = late->alone.out_len; alone.out_bonus = late->alone.out_bonus;
  alone.err = late->alone.err;
  const int b = (int)(blockIdx.x / (unsigned)late->params.W);
  dev::walk_alone<kWideThreads>(alone, b, sh, [&](int r, double& row_max, double& row_z) {
    const float* row = alone.logits + ((long long)b * (alone.n_tree + 1) + r) * alone.vocab;
    float m = -INFINITY;
    for (int v = tid; v < alone.vocab; v += kWideThreads) m = fmaxf(m, row[v]);
    m = dev::block_max_f32<kWideThreads>(m, sh.red);
    row_max = m == -INFINITY ? 0.0 : (double)m / alone.temp;
    double z = 0.0;
    for (int v = tid; v < alone.vocab; v += kWideThreads) z += exp((double)row[v] / alone.temp - row_max);
    row_z = dev::block_sum_f64<kWideThreads>(z, sh.red);
  });
}

}  // namespace

// The blocks of kCoopMaxTrees trees are part of every acceptance workspace, whatever a call's mode and
// batch size: nothing else is ever laid over them, so greedy and sampling calls of any shapes can
// take turns on one workspace without disturbing the words the cooperative walk keeps between calls.
constexpr int kCoopMaxTrees = 512;
size_t accept_coop_bytes() { return (size_t)kCoopMaxTrees * sizeof(TreeBlock); }

unsigned W_reciprocal(int W) { return W > 1 ? (unsigned)((1ull << 32) / (unsigned)W + 1) : 0u; }

template <int PER, int THREADS>
hipError_t launch_walk(const CoopParams& cp, int wgs, hipStream_t stream) {
  if constexpr (PER > 4) return launch_kernel(walk_sample_long_kernel<PER, THREADS>, dim3((unsigned)wgs), dim3(THREADS), 0, stream, cp);
  else return launch_kernel(walk_sample_coop_kernel<PER, THREADS>, dim3((unsigned)wgs), dim3(THREADS), 0, stream, cp.logits, cp.parent, cp.tokens,
                     cp.uniforms, cp.draft_row, cp.n_tree, cp.vocab, cp.W, W_reciprocal(cp.W), cp);
}

template <int PER>
hipError_t launch_wide(CoopParams cp, const dev::AloneParams& alone, int wgs, hipStream_t stream) {
  if (tuning().spin_limit < 0) cp.spin_limit = kWideSpinLimit;
  return launch_kernel(walk_sample_wide_kernel<PER>, dim3((unsigned)wgs), dim3(kWideThreads), 0, stream, cp, alone);
}

bool accept_coop_plan(int batch, int vocab, int cus, int* W, int* slice) {
  if (batch > kCoopMaxTrees) return false;
  auto fits = [&](int threads, int per, int wgs) {
    const int need = (vocab + threads * per - 1) / (threads * per);
    if (need > 64 || (long long)need * batch > wgs || vocab < per) return false;
    *W = need;
    *slice = threads * per;
    return true;
  };
  // Entries per thread: fewer of them mean more workgroups to wait for, more of them longer rows of exponentials.  (us, the mean
  // of six draws, trees x entries: 8 x 32000 with 2 a thread (63 workgroups a tree) 21.6, 4 20.8, 8 23.6; 16 x 32000 with 4 25.1,
  // 8 26.8; 64 x 8000 24.9, 27.6.)  Two only where every workgroup has a CU to itself: 1 x 8000 11.7, with four 12.8; 8 x 8000
  // 17.4 and 19.5.
  if (fits(kCoopThreads, 2, cus)) return true;
  for (int per = 4; per <= 16; per *= 2)
    if (fits(kCoopThreads, per, 2 * cus)) return true;  // (two workgroups of 256 threads per CU are resident together)
  for (int per = 16; per <= 40; per += 8)
    if (fits(kWideThreads, per, cus)) return true;
  return false;
}

hipError_t launch_accept_coop(const AcceptArgs& a, void* coop_ws, double* resid, int W, int slice, hipStream_t stream) {
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
  const dev::AloneParams alone = dev::alone_params(a, resid);
  // A workgroup with a CU to itself has its slice among twice the threads: two waves on a SIMD fill each other's waits.  (us, 256
  // threads / 512: 1 x 128256 16.5 / 15.8, 8 x 32000 20.8 / 20.5; slices of 512 entries 11.7 / 12.0 at 1 x 8000: not those.)
  const bool lone = a.batch * W <= device_cu_count();
  switch (slice) {
    case kCoopThreads * 2: return launch_walk<2, kCoopThreads>(cp, a.batch * W, stream);
    case kCoopThreads * 4: return lone ? launch_walk<2, 512>(cp, a.batch * W, stream) : launch_walk<4, kCoopThreads>(cp, a.batch * W, stream);
    case kCoopThreads * 8: return lone ? launch_walk<4, 512>(cp, a.batch * W, stream) : launch_walk<8, kCoopThreads>(cp, a.batch * W, stream);
    case kCoopThreads * 16: return lone ? launch_walk<8, 512>(cp, a.batch * W, stream) : launch_walk<16, kCoopThreads>(cp, a.batch * W, stream);
    case kWideThreads * 16: return launch_wide<16>(cp, alone, a.batch * W, stream);
    case kWideThreads * 24: return launch_wide<24>(cp, alone, a.batch * W, stream);
    case kWideThreads * 32: return launch_wide<32>(cp, alone, a.batch * W, stream);
    case kWideThreads * 40: return launch_wide<40>(cp, alone, a.batch * W, stream);
    default: return hipErrorInvalidValue;
  }
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
  return launch_kernel(stream_read_kernel, dim3(grid), dim3(256), 0, stream, static_cast<const probe_u32x4*>(src), n,
                     static_cast<unsigned*>(sink));
}

// zero fill as a kernel (safe inside HIP-graph capture, unlike a memset node)
__global__ void zero_fill_kernel(unsigned long long* p, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0ull;
}
hipError_t launch_zero_fill(void* p, size_t bytes, hipStream_t stream) {
  const size_t n = bytes / 8;
  if (n == 0) return hipSuccess;
  const unsigned grid = (unsigned)((n + 255) / 256 < 1024 ? (n + 255) / 256 : 1024);
  return launch_kernel(zero_fill_kernel, dim3(grid), dim3(256), 0, stream, static_cast<unsigned long long*>(p), n);
}

}  // namespace jk
