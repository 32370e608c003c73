// Draft head step of the MoE draft model (gfx950): the two feature rows that the shared output
// embedding sees (Section 3.1.2 Eq. 4: the two selected experts' features scaled by their router
// scores; Section 3.2 Eq. 6-8: their weighted sum and their weighted difference), the logits of
// both heads, the draft distributions q = softmax(logits / temperature) that the acceptance test
// divides by, and each head's top-k candidates.
//
// Kernels:
//   head_inputs_kernel     X[2R, d] bf16 from f_top, s_top (elementwise; more than 32 tokens:
//                          of fewer the product makes its rows itself)
//   row_stats_kernel; row_whole_kernel; row_parts_kernel, row_finish_kernel   per logits row: maximum, normaliser,
//                          top-k by value (ties to the lower token id), probabilities: with the
//                          product's statistics, of short rows, of longer ones.
//   router_kernel, gated_act_kernel, select_kernel   the draft layer's router (Eq. 2, 5) and what
//                          surrounds the experts' three projections (Eq. 3).
// The products with weight matrices run in stream_gemm.hip and ring_gemm.hip.

#include <cfloat>
#include <cmath>
#include <type_traits>

#include "jk_internal.h"
#include "jk_wave.h"

namespace jk {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ unsigned bf16_bits_rne(float f) {
  const unsigned u = __float_as_uint(f);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (u >> 16) | 0x40u;  // NaN stays NaN
  return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}
__device__ __forceinline__ float bf16_lo(unsigned w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(unsigned w) { return __uint_as_float(w & 0xFFFF0000u); }

// ------------------------------------------------------------------ head inputs (Eq. 4 / Eq. 6, 7)
struct MixParams {
  const unsigned short* f_top;  // [rows][2][d] bf16
  const float* s_top;           // [rows][2]
  unsigned short* x;            // [2 rows][d] bf16, row 2r + h
  int rows, d, mode;
  float alpha, beta;
};

// One thread per 8 columns of a token: both heads' rows from one trip to its two features.
__global__ __launch_bounds__(64) void head_inputs_kernel(MixParams p) {
  const int d8 = p.d / 8;
  const long long i = (long long)blockIdx.x * 64 + threadIdx.x;
  if (i >= (long long)p.rows * d8) return;
  const int r = (int)(i / d8), c = (int)(i % d8);
  const u32x4 a = reinterpret_cast<const u32x4*>(p.f_top + ((long long)r * 2 + 0) * p.d)[c];
  const u32x4 b = reinterpret_cast<const u32x4*>(p.f_top + ((long long)r * 2 + 1) * p.d)[c];
  const float s1 = p.s_top[2 * r], s2 = p.s_top[2 * r + 1];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    // x = c1 f1 + c2 f2
    float c1, c2;
    if (p.mode == JK_HEADS_DECOUPLED) {
      c1 = h == 0 ? s1 : 0.f;
      c2 = h == 0 ? 0.f : s2;
    } else {
      c1 = h == 0 ? s1 : p.beta;
      c2 = h == 0 ? s2 : -p.alpha;
    }
    u32x4 o;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      // a term whose coefficient is zero is left out, so that a NaN in the other expert's
      // feature cannot leak into a decoupled head
      const float lo = (c1 != 0.f ? c1 * bf16_lo(a[j]) : 0.f) + (c2 != 0.f ? c2 * bf16_lo(b[j]) : 0.f);
      const float hi = (c1 != 0.f ? c1 * bf16_hi(a[j]) : 0.f) + (c2 != 0.f ? c2 * bf16_hi(b[j]) : 0.f);
      o[j] = bf16_bits_rne(lo) | (bf16_bits_rne(hi) << 16);
    }
    reinterpret_cast<u32x4*>(p.x + (long long)(2 * r + h) * p.d)[c] = o;
  }
}

// ------------------------------------------------------------------ softmax + top-k per logits row
// A row (a vocabulary of 10^5 entries) is cut into parts of 256 threads x PT entries so that the work spreads over all
// CUs; everything a thread needs is in its registers after one trip to memory:
//   row_parts_kernel   per (row, part): maximum, sum of exp((x - max) / T), the part's k best
//   row_whole_kernel   all of it, for short rows: one workgroup of 1024 threads per row
//   row_stats_kernel   what row_finish_kernel does, where the product has left the statistics of each row's 128 entries
//   row_finish_kernel  a workgroup per row first: the k best of the parts' candidates, their probabilities; then one per
//                      (row, part): q = exp((x - max) / T) / Z (if asked for).  Each takes the row's maximum and
//                      normaliser from the parts' pairs for itself.
constexpr int kPartThreads = 256;
constexpr int kPartPerThreadMax = 16;
constexpr int kMaxTopK = 16;

struct SoftParams {
  float* logits;        // [n_rows][vocab]
  const float* sums;    // or null: [ksplit][n_rows][vocab] partial logits, summed up here
  int ksplit;
  float* probs;         // [n_rows][vocab] or nullptr
  int* tk_ids;          // [n_rows][k]
  float* tk_probs;      // [n_rows][k]
  float* part_ms;       // [n_rows][parts][2]   max, sum
  unsigned long long* keys;  // [n_rows][parts][k]   candidates, best first (0: none)
  int n_rows, vocab, k, parts, part_len;  // part_len: entries per part, a multiple of 4
  float inv_temp;
  const float2* stats;  // row_stats_kernel: [n_rows][blocks] (maximum, sum) of kStatColumns entries each, from the product
  int blocks;
  float scale_hi, scale_lo;  // (see StreamGemmArgs)
};

// Order of candidates - larger value first, equal values by increasing id - as one unsigned comparison: the value's bits
// made monotonic (+ 0: the two zeros are equal) above the complement of the id.  No candidate has key 0.
__device__ __forceinline__ unsigned ordered_bits(float v) {
  const unsigned u = __float_as_uint(v + 0.f);
  return u ^ ((u >> 31) ? 0xFFFFFFFFu : 0x80000000u);
}
__device__ __forceinline__ unsigned long long key_of(float v, int id) {
  return ((unsigned long long)ordered_bits(v) << 32) | (unsigned)~id;
}
__device__ __forceinline__ int key_id(unsigned long long k) { return (int)~(unsigned)k; }
__device__ __forceinline__ float key_value(unsigned long long k) {
  const unsigned u = (unsigned)(k >> 32);
  return __uint_as_float(u ^ ((u >> 31) ? 0x80000000u : 0xFFFFFFFFu));
}
__device__ __forceinline__ unsigned long long wave_max_key(unsigned long long k) {  // (see jk_wave.h)
  auto most = [&](unsigned lo, unsigned hi) {
    const unsigned long long other = (unsigned long long)hi << 32 | lo;
    k = other > k ? other : k;
  };
  auto lo = [&] { return (unsigned)k; };
  auto hi = [&] { return (unsigned)(k >> 32); };
  most((unsigned)dev::dpp<0xB1>((int)lo()), (unsigned)dev::dpp<0xB1>((int)hi()));    // quad_perm [1,0,3,2]
  most((unsigned)dev::dpp<0x4E>((int)lo()), (unsigned)dev::dpp<0x4E>((int)hi()));    // quad_perm [2,3,0,1]
  most((unsigned)dev::dpp<0x141>((int)lo()), (unsigned)dev::dpp<0x141>((int)hi()));  // row_half_mirror
  most((unsigned)dev::dpp<0x140>((int)lo()), (unsigned)dev::dpp<0x140>((int)hi()));  // row_mirror
  const int lane = __lane_id();
  most(dev::other16(lo(), lane & 16), dev::other16(hi(), lane & 16));
  most(dev::other32(lo(), lane & 32), dev::other32(hi(), lane & 32));
  return k;
}

constexpr int kCandCap = 512;

// Place of each of the n listed keys (all different) by counting the larger ones: `put(rank, key)` for ranks below k.
template <int THREADS = kPartThreads, class F>
__device__ __forceinline__ void rank_list(const unsigned long long* list, int n, int k, F put) {
  for (int j = threadIdx.x; j < n; j += THREADS) {
    const unsigned long long mine = list[j];
    int rank = 0;
#pragma unroll 8
    for (int i = 0; i < n; ++i) rank += (int)(list[i] > mine);
    if (rank < k) put(rank, mine);
  }
}

// The k-th largest of a wave's 64 values (k at most 64): the least of the values that fewer than k others exceed.  Ranking
// by reading every lane in turn needs no memory and no rounds.
__device__ __forceinline__ float wave_kth_largest(float v, int k) {
  int above = 0;
#pragma unroll
  for (int j = 0; j < 64; ++j) above += (int)(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), j)) > v);
  return -dev::wave_max(above < k ? -v : -INFINITY);
}

// A part as its workgroup holds it: PT entries a thread, ids increasing with the index.  Four consecutive entries per
// load where rows start at multiples of 16 bytes, single ones otherwise; past the end: -inf.
template <int PT, int THREADS = kPartThreads>
struct PartView {
  int lo, hi, tid;
  bool vec;
  __device__ __forceinline__ PartView(const SoftParams& p, int part, bool aligned)
      : lo(part * p.part_len), hi(min(p.vocab, part * p.part_len + p.part_len)), tid(threadIdx.x), vec(aligned && (p.vocab & 3) == 0) {}
  __device__ __forceinline__ int id(int i) const {
    return lo + (vec ? 4 * (tid + THREADS * (i >> 2)) + (i & 3) : tid + THREADS * i);
  }
  __device__ __forceinline__ void load(const float* x, float (&val)[PT]) const {
    if (vec) {
#pragma unroll
      for (int u = 0; u < PT / 4; ++u) {
        const int e = lo + 4 * (tid + THREADS * u);
        floatx4 q = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
        if (e < hi) q = *reinterpret_cast<const floatx4*>(x + e);
#pragma unroll
        for (int c = 0; c < 4; ++c) val[4 * u + c] = q[c];
      }
    } else {
#pragma unroll
      for (int i = 0; i < PT; ++i) {
        const int e = lo + tid + THREADS * i;
        val[i] = e < hi ? x[e] : -INFINITY;
      }
    }
  }
  __device__ __forceinline__ void store(float* x, const float (&val)[PT]) const {
    if (vec) {
#pragma unroll
      for (int u = 0; u < PT / 4; ++u) {
        const int e = lo + 4 * (tid + THREADS * u);
        if (e < hi) *reinterpret_cast<floatx4*>(x + e) = floatx4{val[4 * u], val[4 * u + 1], val[4 * u + 2], val[4 * u + 3]};
      }
    } else {
#pragma unroll
      for (int i = 0; i < PT; ++i) {
        const int e = lo + tid + THREADS * i;
        if (e < hi) x[e] = val[i];
      }
    }
  }
};
__device__ __forceinline__ bool on16(const void* p) { return (reinterpret_cast<size_t>(p) & 15) == 0; }

// A part's logits; the k parts' partial products come together here, in a fixed order
template <int PT, class View>
__device__ __forceinline__ void load_logits(const SoftParams& p, const View& view, int row, float (&val)[PT]) {
  const long long at = (long long)row * p.vocab;
  if (p.sums) {
    const long long step = (long long)p.n_rows * p.vocab;
    view.load(p.sums + at, val);
    constexpr int kAhead = PT <= 4 ? 4 : (PT <= 8 ? 2 : 1);
#pragma unroll kAhead
    for (int z = 1; z < p.ksplit; ++z) {
      float more[PT];
      view.load(p.sums + at + z * step, more);
#pragma unroll
      for (int i = 0; i < PT; ++i) val[i] += more[i];
    }
    view.store(p.logits + at, val);
  } else {
    view.load(p.logits + at, val);
  }
}

// Top-k of a part: the k-th largest of 64 disjoint groups' maxima is a lower bound of the part's
// k-th largest value, so only entries at or above it can be among the k best; they are put on a
// short list in LDS (few, unless the part is full of ties) and each listed entry finds its place
// by counting the entries that beat it.  A part with more such entries than the list holds
// takes k passes over the registers instead.
template <int PT>
__global__ __launch_bounds__(kPartThreads) void row_parts_kernel(SoftParams p) {
  __shared__ unsigned long long cand[kCandCap];
  __shared__ unsigned long long sk[2][4];
  __shared__ float lane_max[kPartThreads];
  __shared__ float sf[4], ss[4];
  __shared__ float s_tau;
  __shared__ int n_cand;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, V = p.vocab, K = p.k;
  const int row = blockIdx.x / p.parts, part = blockIdx.x % p.parts;
  const PartView<PT> view(p, part, on16(p.logits) && on16(p.sums));
  float val[PT];
  load_logits<PT>(p, view, row, val);
  float tv = -INFINITY;
#pragma unroll
  for (int i = 0; i < PT; ++i) tv = fmaxf(tv, val[i]);
  lane_max[tid] = tv;
  {
    const float m = dev::wave_max(tv);
    if (lane == 0) sf[wave] = m;
  }
  if (tid == 0) n_cand = 0;
  __syncthreads();
  const float m = fmaxf(fmaxf(sf[0], sf[1]), fmaxf(sf[2], sf[3]));
  const float m_use = m > -INFINITY ? m : 0.f;  // a part of -inf only: nothing sensible to subtract
  if (wave == 0) {  // the threshold: group g is threads g, g + 64, ...
    const float t = wave_kth_largest(fmaxf(fmaxf(tv, lane_max[lane + 64]), fmaxf(lane_max[lane + 128], lane_max[lane + 192])), K);
    if (lane == 0) s_tau = t;
  }
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < PT; ++i) s += expf((val[i] - m_use) * p.inv_temp);
  s = dev::wave_sum(s);
  if (lane == 0) ss[wave] = s;
  __syncthreads();
  const long long slot = (long long)row * p.parts + part;
  if (tid == 0) {
    p.part_ms[2 * slot] = m;
    p.part_ms[2 * slot + 1] = (ss[0] + ss[1]) + (ss[2] + ss[3]);
  }
  const float tau = s_tau;
#pragma unroll
  for (int i = 0; i < PT; ++i)
    if (val[i] >= tau && val[i] > -INFINITY) {  // (-inf: past the end, or impossible)
      const int at = atomicAdd(&n_cand, 1);
      if (at < kCandCap) cand[at] = key_of(val[i], view.id(i));
    }
  __syncthreads();
  const int nc = n_cand;
  unsigned long long* out = p.keys + slot * K;
  if (nc <= kCandCap) {
    if (tid < K && tid >= nc) out[tid] = 0ull;  // (a part with fewer than k entries)
    rank_list(cand, nc, K, [&](int rank, unsigned long long key) { out[rank] = key; });
  } else {
    // one winner per pass: the largest key below the previous winner's
    unsigned long long prev = ~0ull;
    for (int round = 0; round < K; ++round) {
      unsigned long long best = 0ull;
#pragma unroll
      for (int i = 0; i < PT; ++i) {
        const unsigned long long key = key_of(val[i], view.id(i));
        if (val[i] >= tau && val[i] > -INFINITY && key < prev && key > best) best = key;
      }
      best = wave_max_key(best);
      if (lane == 0) sk[round & 1][wave] = best;
      __syncthreads();  // (one is enough: the buffers alternate)
#pragma unroll
      for (int w = 0; w < 4; ++w) best = sk[round & 1][w] > best ? sk[round & 1][w] : best;
      if (tid == 0) out[round] = best;  // 0 once the part is exhausted: nothing comes after it
      prev = best;
    }
  }
}

// The row's maximum and 1 / normaliser from the parts' (max, sum) pairs, and (for the top-k) the k-th largest of 64
// groups of parts' maxima: every wave of every workgroup that needs them reduces the pairs for itself, the same operations
// in the same order everywhere.
__device__ __forceinline__ void row_max_and_norm(const SoftParams& p, int row, float& m_use, float& inv_z, float& group_max) {
  const int lane = threadIdx.x & 63, P = p.parts;
  const float2* ms = reinterpret_cast<const float2*>(p.part_ms) + (long long)row * P;
  float2 own = make_float2(-INFINITY, 0.f);  // (rarely more than one part per lane)
  if (lane < P) own = ms[lane];
  float m = own.x;
  for (int i = lane + 64; i < P; i += 64) m = fmaxf(m, ms[i].x);
  group_max = m;
  m = dev::wave_max(m);
  m_use = m > -INFINITY ? m : 0.f;
  double z = own.x > -INFINITY ? (double)own.y * (double)expf((own.x - m_use) * p.inv_temp) : 0.0;
  for (int i = lane + 64; i < P; i += 64) {
    const float2 q = ms[i];
    if (q.x > -INFINITY) z += (double)q.y * (double)expf((q.x - m_use) * p.inv_temp);
  }
  inv_z = (float)(1.0 / dev::wave_sum(z));
}

// The k best of the parts' candidates and their probabilities (one workgroup of four waves per row).  As in a part: the
// k-th largest of 64 groups' maxima bounds the row's k-th best from below, and few candidates reach it.
__device__ __forceinline__ void row_top_k(const SoftParams& p, int row) {
  __shared__ unsigned long long cand[kCandCap];
  __shared__ int n_cand;
  const int tid = threadIdx.x, lane = tid & 63, K = p.k, n = p.parts * K;
  const unsigned long long* keys = p.keys + (long long)row * n;
  if (tid == 0) n_cand = 0;
  __syncthreads();
  float m, inv_z, groups;
  row_max_and_norm(p, row, m, inv_z, groups);
  const unsigned tau = ordered_bits(wave_kth_largest(groups, K));
#pragma unroll 4
  for (int i = tid; i < n; i += kPartThreads) {
    const unsigned long long key = keys[i];
    if (key != 0ull && (unsigned)(key >> 32) >= tau) {
      const int at = atomicAdd(&n_cand, 1);
      if (at < kCandCap) cand[at] = key;
    }
  }
  __syncthreads();
  const int nc = n_cand;
  auto put = [&](int rank, unsigned long long key) {
    p.tk_ids[(long long)row * K + rank] = key_id(key);
    p.tk_probs[(long long)row * K + rank] = expf((key_value(key) - m) * p.inv_temp) * inv_z;
  };
  auto put_none = [&](int rank) {  // fewer than k candidates in the whole row
    p.tk_ids[(long long)row * K + rank] = 0;
    p.tk_probs[(long long)row * K + rank] = 0.f;
  };
  if (nc <= kCandCap) {
    if (tid < K && tid >= nc) put_none(tid);
    rank_list(cand, nc, K, put);
    return;
  }
  if (tid >= 64) return;  // very many ties: one wave, k selection passes over the candidates in memory
  unsigned long long prev = ~0ull;
  for (int round = 0; round < K; ++round) {
    unsigned long long best = 0ull;
    for (int i = lane; i < n; i += 64) {
      const unsigned long long key = keys[i];
      if (key < prev && key > best) best = key;
    }
    best = wave_max_key(best);
    if (lane == 0) {
      if (best != 0ull) put(round, best);
      else put_none(round);
    }
    prev = best;
  }
}

template <int PT>
__global__ __launch_bounds__(kPartThreads) void row_finish_kernel(SoftParams p) {
  const int V = p.vocab;
  if ((int)blockIdx.x < p.n_rows) {  // (the longer chain: started first)
    row_top_k(p, blockIdx.x);
    return;
  }
  const int at = (int)blockIdx.x - p.n_rows, row = at / p.parts, part = at % p.parts;
  const PartView<PT> view(p, part, on16(p.logits) && on16(p.probs));
  float val[PT], m, inv_z, groups;
  view.load(p.logits + (long long)row * V, val);  // on its way while the row's pairs are reduced
  row_max_and_norm(p, row, m, inv_z, groups);
#pragma unroll
  for (int i = 0; i < PT; ++i) val[i] = expf((val[i] - m) * p.inv_temp) * inv_z;
  view.store(p.probs + (long long)row * V, val);
}

// ---- The product's workgroups leave the (maximum, sum) of each row's blocks of 128 entries, which are in their LDS for the result's sake: no
// launch that reads all logits for them.  A workgroup of four waves takes a row's maximum and normaliser from the pairs, the
// same operations in the same order everywhere.
struct RowStats {
  float m, inv_z;
  float2 own[4];  // this thread's first blocks: tid, tid + 256, ...
};
struct RowStatsShared {
  float top[4];
  double sum[4];
  float lane_max[kPartThreads];
  float tau;
};
// LIST: also the k-th largest of 64 groups of blocks' maxima, in sh.tau (behind the caller's next barrier too)
template <bool LIST>
__device__ __forceinline__ RowStats row_stats(const SoftParams& p, const float2* ms, RowStatsShared& sh) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  RowStats s;
  float top = -INFINITY;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int j = tid + kPartThreads * u;
    s.own[u] = make_float2(-INFINITY, 0.f);
    if (j < p.blocks) s.own[u] = ms[j];
    top = fmaxf(top, s.own[u].x);
  }
  for (int j = tid + 4 * kPartThreads; j < p.blocks; j += kPartThreads) top = fmaxf(top, ms[j].x);
  if (LIST) sh.lane_max[tid] = top;
  top = dev::wave_max(top);
  if (lane == 0) sh.top[wave] = top;
  __syncthreads();
  const float m = fmaxf(fmaxf(sh.top[0], sh.top[1]), fmaxf(sh.top[2], sh.top[3]));
  s.m = m > -INFINITY ? m : 0.f;
  double z = 0.0;  // (a block of -inf only: 0 times 0; of NaNs: NaN)
  auto add = [&](float2 q) { z += (double)q.y * (double)dev::exp_scaled(q.x - s.m, p.scale_hi, p.scale_lo); };
#pragma unroll
  for (int u = 0; u < 4; ++u) add(s.own[u]);
  for (int j = tid + 4 * kPartThreads; j < p.blocks; j += kPartThreads) add(ms[j]);
  z = dev::wave_sum(z);
  if (lane == 0) sh.sum[wave] = z;
  if (LIST && wave == 0) {
    const float t = wave_kth_largest(fmaxf(fmaxf(sh.lane_max[lane], sh.lane_max[lane + 64]), fmaxf(sh.lane_max[lane + 128], sh.lane_max[lane + 192])), p.k);
    if (lane == 0) sh.tau = t;
  }
  __syncthreads();
  s.inv_z = (float)(1.0 / ((sh.sum[0] + sh.sum[1]) + (sh.sum[2] + sh.sum[3])));
  return s;
}

// The k best of a row: entries at or above the threshold, all in blocks whose maximum is; few blocks, and few entries, unless
// there are many ties.  Then k rounds, each the largest key below the last winner's: of a block with no winner yet, its
// maximum at its first place stands for its best key; the others, at most as many as there were winners, are looked through.
__device__ __forceinline__ void row_stats_top_k(const SoftParams& p, int row) {
  constexpr int kListed = 256;
  __shared__ RowStatsShared sh;
  __shared__ unsigned long long cand[kCandCap], sk[2][4];
  __shared__ int list[kListed];
  __shared__ int n_list, n_cand;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, K = p.k;
  const float2* ms = p.stats + (long long)row * p.blocks;
  const float* x = p.logits + (long long)row * p.vocab;
  if (tid == 0) n_list = n_cand = 0;
  const RowStats s = row_stats<true>(p, ms, sh);
  auto put = [&](int rank, unsigned long long key) {  // (0: fewer than k candidates in the whole row)
    p.tk_ids[(long long)row * K + rank] = key ? key_id(key) : 0;
    p.tk_probs[(long long)row * K + rank] = key ? expf((key_value(key) - s.m) * p.inv_temp) * s.inv_z : 0.f;
  };
  auto entry = [&](int block, int e) {  // (past the end: -inf, as an impossible one)
    const int i = block * kStatColumns + e;
    return i < p.vocab ? x[i] : -INFINITY;
  };
  const float tau = sh.tau;
  auto look = [&](int j, float top) {
    if (!(top >= tau && top > -INFINITY)) return;
    const int at = atomicAdd(&n_list, 1);
    if (at < kListed) list[at] = j;
  };
#pragma unroll
  for (int u = 0; u < 4; ++u) look(tid + kPartThreads * u, s.own[u].x);
  for (int j = tid + 4 * kPartThreads; j < p.blocks; j += kPartThreads) look(j, ms[j].x);
  __syncthreads();
  const int listed = n_list;
  if (listed <= kListed) {
    constexpr int AT_ONCE = 4;
    for (int i0 = wave; i0 < listed; i0 += 4 * AT_ONCE) {
      int block[AT_ONCE];
      float v[AT_ONCE][2];
#pragma unroll
      for (int u = 0; u < AT_ONCE; ++u) {  // (one past the list's end: its last once more, and not used)
        block[u] = list[min(i0 + 4 * u, listed - 1)];
        v[u][0] = entry(block[u], lane);
        v[u][1] = entry(block[u], lane + 64);
      }
#pragma unroll
      for (int u = 0; u < AT_ONCE; ++u)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          if (i0 + 4 * u < listed && v[u][h] >= tau && v[u][h] > -INFINITY) {
            const int at = atomicAdd(&n_cand, 1);
            if (at < kCandCap) cand[at] = key_of(v[u][h], block[u] * kStatColumns + lane + 64 * h);
          }
    }
    __syncthreads();
    const int nc = n_cand;
    if (nc <= kCandCap) {
      if (tid < K && tid >= nc) put(tid, 0ull);
      rank_list(cand, nc, K, put);
      return;
    }
  }
  unsigned long long prev = ~0ull;
  for (int round = 0; round < K; ++round) {
    __syncthreads();  // (the list of the round before has been read)
    if (tid == 0) n_list = 0;
    __syncthreads();
    unsigned long long best = 0ull;
    for (int j = tid; j < p.blocks; j += kPartThreads) {
      const float top = ms[j].x;
      if (!(top > -INFINITY)) continue;
      const unsigned long long first = key_of(top, j * kStatColumns);  // (none of the block's keys is larger)
      if (first < prev) {
        best = first > best ? first : best;
      } else {
        const int at = atomicAdd(&n_list, 1);
        if (at < kListed) list[at] = j;
      }
    }
    __syncthreads();
    for (int i = wave; i < min(n_list, kListed); i += 4)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const float v = entry(list[i], lane + 64 * h);
        const unsigned long long key = key_of(v, list[i] * kStatColumns + lane + 64 * h);
        if (v > -INFINITY && key < prev && key > best) best = key;
      }
    best = wave_max_key(best);
    if (lane == 0) sk[round & 1][wave] = best;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < 4; ++w) best = sk[round & 1][w] > best ? sk[round & 1][w] : best;
    if (best != 0ull) {
      const int j = key_id(best) / kStatColumns;
      if (key_of(ms[j].x, j * kStatColumns) == best) {  // (a block without a winner: where its maximum is)
        const unsigned want = (unsigned)(best >> 32);
        const unsigned long long lo = __ballot(ordered_bits(entry(j, lane)) == want), hi = __ballot(ordered_bits(entry(j, lane + 64)) == want);
        best = (best & ~0xFFFFFFFFull) | (unsigned)~(j * kStatColumns + (lo ? __ffsll((long long)lo) - 1 : 63 + __ffsll((long long)hi)));
      }
    }
    if (tid == 0) put(round, best);
    if (best == 0ull) {  // (nothing comes after it)
      if (tid > round && tid < K) put(tid, 0ull);
      return;
    }
    prev = best;
  }
}

// Bound by the trips to memory of its longer chain (the k best: pairs, blocks that matter, their entries), which starts first.
// 20 rows of 128256: 9.4 us under the tracer, 7.2 without the distributions, where the two launches took 7.05 and 6.95.
template <int PT>
__global__ __launch_bounds__(kPartThreads) void row_stats_kernel(const float2* stats, float* logits, int n_rows, int parts, int blocks, int vocab, int part_len,
                                                                 int k, float* probs, SoftParams p) {
  p.stats = stats; p.logits = logits; p.probs = probs;
  p.n_rows = n_rows; p.parts = parts; p.blocks = blocks; p.vocab = vocab; p.part_len = part_len; p.k = k;
  if ((int)blockIdx.x < p.n_rows) {
    row_stats_top_k(p, blockIdx.x);
    return;
  }
  __shared__ RowStatsShared sh;
  const int at = (int)blockIdx.x - p.n_rows, row = at / p.parts, part = at % p.parts;
  const PartView<PT> view(p, part, on16(p.logits) && on16(p.probs));
  float val[PT];
  view.load(p.logits + (long long)row * p.vocab, val);  // on its way while the row's pairs are reduced
  const RowStats s = row_stats<false>(p, p.stats + (long long)row * p.blocks, sh);
#pragma unroll
  for (int i = 0; i < PT; ++i) val[i] = expf((val[i] - s.m) * p.inv_temp) * s.inv_z;
  view.store(p.probs + (long long)row * p.vocab, val);
}

// A short row whole: a workgroup of 16 waves has it in its registers, so that nothing is left for a second launch and no logit
// is read twice.  The second launch was 2 - 4 us of 12 - 30 (calls of 1024 columns, us, before / now: 4 tokens and 4000 entries 14.9 /
// 11.7, 8000 13.9 / 11.7; 64 tokens and 16 384 entries 30.5 / 26.5).
constexpr int kRowThreads = 1024, kRowWaves = kRowThreads / 64, kRowPerThreadMax = 32;

template <int PT>
__global__ __launch_bounds__(kRowThreads) void row_whole_kernel(SoftParams p) {
  __shared__ unsigned long long cand[kCandCap];
  __shared__ unsigned long long sk[2][kRowWaves];
  __shared__ float lane_max[kRowThreads];
  __shared__ float sf[kRowWaves], ss[kRowWaves];
  __shared__ float s_tau;
  __shared__ int n_cand;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, V = p.vocab, K = p.k, row = blockIdx.x;
  const PartView<PT, kRowThreads> view(p, 0, on16(p.logits) && on16(p.sums) && on16(p.probs));
  float val[PT], e[PT];
  load_logits<PT>(p, view, row, val);
  float tv = -INFINITY;
#pragma unroll
  for (int i = 0; i < PT; ++i) tv = fmaxf(tv, val[i]);
  lane_max[tid] = tv;
  {
    const float m = dev::wave_max(tv);
    if (lane == 0) sf[wave] = m;
  }
  if (tid == 0) n_cand = 0;
  __syncthreads();
  const float m = dev::wave_max(sf[lane & (kRowWaves - 1)]);
  const float m_use = m > -INFINITY ? m : 0.f;
  if (wave == 0) {  // the threshold: group g is threads g, g + 64, ...
    float t = tv;
#pragma unroll
    for (int w = 1; w < kRowWaves; ++w) t = fmaxf(t, lane_max[lane + 64 * w]);
    t = wave_kth_largest(t, K);
    if (lane == 0) s_tau = t;
  }
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < PT; ++i) s += e[i] = expf((val[i] - m_use) * p.inv_temp);
  s = dev::wave_sum(s);
  if (lane == 0) ss[wave] = s;
  __syncthreads();
  const float inv_z = (float)(1.0 / dev::wave_sum(lane < kRowWaves ? (double)ss[lane] : 0.0));
  const float tau = s_tau;
#pragma unroll
  for (int i = 0; i < PT; ++i)
    if (val[i] >= tau && val[i] > -INFINITY) {  // (-inf: past the end, or impossible)
      const int at = atomicAdd(&n_cand, 1);
      if (at < kCandCap) cand[at] = key_of(val[i], view.id(i));
    }
  if (p.probs) {
#pragma unroll
    for (int i = 0; i < PT; ++i) e[i] *= inv_z;
    view.store(p.probs + (long long)row * V, e);
  }
  __syncthreads();
  const int nc = n_cand;
  auto put = [&](int rank, unsigned long long key) {  // (0: fewer than k candidates)
    p.tk_ids[(long long)row * K + rank] = key ? key_id(key) : 0;
    p.tk_probs[(long long)row * K + rank] = key ? expf((key_value(key) - m_use) * p.inv_temp) * inv_z : 0.f;
  };
  if (nc <= kCandCap) {
    if (tid < K && tid >= nc) put(tid, 0ull);
    rank_list<kRowThreads>(cand, nc, K, put);
    return;
  }
  unsigned long long prev = ~0ull;  // very many ties: the largest key below the previous winner's per pass
  for (int round = 0; round < K; ++round) {
    unsigned long long best = 0ull;
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      const unsigned long long key = key_of(val[i], view.id(i));
      if (val[i] >= tau && val[i] > -INFINITY && key < prev && key > best) best = key;
    }
    best = wave_max_key(best);
    if (lane == 0) sk[round & 1][wave] = best;
    __syncthreads();  // (one is enough: the buffers alternate)
#pragma unroll
    for (int w = 0; w < kRowWaves; ++w) best = sk[round & 1][w] > best ? sk[round & 1][w] : best;
    if (tid == 0) put(round, best);
    prev = best;
  }
}

template <int PT>
hipError_t launch_rows(const SoftParams& p, hipStream_t stream) {
  const unsigned parts = (unsigned)(p.n_rows * p.parts);
  if (p.stats) {
    return launch_kernel(row_stats_kernel<PT>, dim3(p.n_rows + (p.probs ? parts : 0u)), dim3(kPartThreads), 0, stream, p.stats, p.logits, p.n_rows, p.parts, p.blocks,
                       p.vocab, p.part_len, p.k, p.probs, p);
  }
  hipLaunchKernelGGL(row_parts_kernel<PT>, dim3(parts), dim3(kPartThreads), 0, stream, p);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  return launch_kernel(row_finish_kernel<PT>, dim3(p.n_rows + (p.probs ? parts : 0u)), dim3(kPartThreads), 0, stream, p);
}

// Rows of up to 16 entries a thread whole; longer ones only where there are so many that parts would not spread them over more CUs (what a
// CU draws bounds the kernel then).  Calls of 1024 columns, us, in parts / whole: 1 token and 16 384 entries 16.3 / 16.0, 24 000 17.6 / 19.9, 32 000
// 20.5 / 22.5; 10 tokens 17.8 / 17.1, 19.9 / 21.9, 22.3 / 23.5; 32 tokens 21.7 / 19.6, 23.9 / 23.1, 27.1 / 25.5.
bool rows_whole(int n_rows, int vocab) { return vocab <= kRowThreads * (n_rows >= 64 ? kRowPerThreadMax : kRowPerThreadMax / 2); }

// ------------------------------------------------------------------ router and experts (Eq. 2, 3, 5)
constexpr int kMaxExperts = 64;

// One workgroup per row: the router scores s_j = softmax_j(u . e_j) (Eq. 2; fp32), of which it picks the two largest
// (Eq. 5, K = 2, ties to the lower expert; a NaN score ranks below every other, so that the row always names two
// different experts that exist - the experts' outputs are addressed with them).  Bound by a trip to memory: a wave asks for up to
// 8 KB of the row and of two centroids together (left alone, the compiler asked for one 1 KB piece after the other: 40
// rows of 4096, eight experts, 7.8 us, and 4.9 like this; of the whole call 153.6 and 151.0, of a small one - 64 rows of 1024,
// four experts of 2048 - 29.0 and 29.4), and the softmax and both maxima are taken across the
// lanes of a wave, by lane moves.  (By shuffles, and with eight pieces whatever the row's length; and select_kernel with its
// scores asked for, and waited for, in front of the results: 18 drawn calls of experts 1.036 times as long, small ones 1.04 - 1.09.)
// u [rows][d] and centroids [n_experts][d] bf16, s_top and idx [rows][2].  (These kernels' arguments are in scalar registers when a wave
// starts, a compiler option for this file, fourteen words at most: from memory they took 0.3 us of each.  Calls, us, so / like this: 8 rows,
// eight experts of 512 x 512 14.2 / 13.9, 64 rows, four of 1024 x 2048 28.8 / 28.0, 40 rows, eight of 4096 x 4096 144.2 / 143.7; heads of one token,
// 30000 x 512 14.4 / 13.8.)
__global__ __launch_bounds__(256) void router_kernel(const uint16_t* u_rows, const uint16_t* centroids, int d, int n_experts, float* s_top, int* idx) {
  __shared__ float score[kMaxExperts];
  const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const u32x4* src = reinterpret_cast<const u32x4*>(u_rows + (long long)row * d);
  // (as many pieces of 1 KB a time as a row has: 2, 4 or 8)
  auto scores = [&](auto n_pieces) {
    for (int j0 = wave; j0 < n_experts; j0 += 8) {  // two experts per pass: their loads share the trip to memory
      const bool two = j0 + 4 < n_experts;
      const u32x4* e0 = reinterpret_cast<const u32x4*>(centroids + (long long)j0 * d);
      const u32x4* e1 = reinterpret_cast<const u32x4*>(centroids + (long long)(two ? j0 + 4 : j0) * d);
      float acc0 = 0.f, acc1 = 0.f;
      constexpr int PIECES = decltype(n_pieces)::value;
      for (int c0 = 0; c0 < d / 8; c0 += 64 * PIECES) {
        u32x4 a[PIECES], b0[PIECES], b1[PIECES];
#pragma unroll
        for (int u = 0; u < PIECES; ++u) {
          const int c = min(c0 + 64 * u + lane, d / 8 - 1);
          a[u] = src[c];
          b0[u] = e0[c];
          b1[u] = e1[c];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < PIECES; ++u) {
          if (c0 + 64 * u + lane >= d / 8) break;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            acc0 += bf16_lo(a[u][i]) * bf16_lo(b0[u][i]) + bf16_hi(a[u][i]) * bf16_hi(b0[u][i]);
            acc1 += bf16_lo(a[u][i]) * bf16_lo(b1[u][i]) + bf16_hi(a[u][i]) * bf16_hi(b1[u][i]);
          }
        }
      }
      acc0 = dev::wave_sum(acc0);
      acc1 = dev::wave_sum(acc1);
      if (lane == 0) {
        score[j0] = acc0;
        if (two) score[j0 + 4] = acc1;
      }
    }
  };
  if (d <= 1024) scores(std::integral_constant<int, 2>());
  else if (d <= 2048) scores(std::integral_constant<int, 4>());
  else scores(std::integral_constant<int, 8>());
  __syncthreads();
  if (wave != 0) return;
  // (at most 64 experts; a lane without one has key 0, which loses to every expert's key, a NaN's 0 above ~id included)
  const float mine = lane < n_experts ? score[lane] : -INFINITY;
  const unsigned long long key = lane >= n_experts ? 0ull : mine == mine ? key_of(mine, lane) : (unsigned long long)(unsigned)~lane;
  const int i1 = key_id(wave_max_key(key)), i2 = key_id(wave_max_key(lane == i1 ? 0ull : key));
  auto score_of = [&](int i) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(mine), __builtin_amdgcn_readfirstlane(i))); };
  const float v1 = score_of(i1), v2 = score_of(i2);
  const float z = dev::wave_sum(lane < n_experts ? expf(mine - v1) : 0.f);
  if (lane == 0) {
    s_top[2 * row] = 1.f / z;
    s_top[2 * row + 1] = expf(v2 - v1) / z;
    idx[2 * row] = i1;
    idx[2 * row + 1] = i2;
  }
}

// The k parts' partial results of four consecutive outputs, up to eight of them in flight, added in a fixed order
__device__ __forceinline__ floatx4 sum_parts(const float* part, int ksplit, long long step) {
  floatx4 v = {0.f, 0.f, 0.f, 0.f};
  for (int z0 = 0; z0 < ksplit; z0 += 8) {
    floatx4 t[8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (z0 + i < ksplit) t[i] = *reinterpret_cast<const floatx4*>(part + (z0 + i) * step);
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (z0 + i < ksplit) v += t[i];
  }
  return v;
}

// The same of two results, both in flight together.  What calls this is bound by trips to memory, of which there is one: the
// rows of the experts' results are numbered by choice, so that nothing has to be looked up first, and a thread has one
// quad.  (Numbered expert by expert there were three in a row for select_kernel, and in gated_act_kernel two for each of up to
// four quads.  The whole call, 40 rows and 8 experts of 4096 x 4096: 151.0 us, 149.8 like this; 68 rows, 5 of 3456 x 1536, with a
// divided k range: 57.6 and 53.6; of 36 shapes all faster, 3 % in the mean.)
__device__ __forceinline__ void sum_two(const float* pa, const float* pb, int ksplit, long long step, floatx4& a, floatx4& b) {
  a = b = floatx4{0.f, 0.f, 0.f, 0.f};
  for (int z0 = 0; z0 < ksplit; z0 += 8) {
    floatx4 t[8], u[8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (z0 + i < ksplit) {
        t[i] = *reinterpret_cast<const floatx4*>(pa + (z0 + i) * step);
        u[i] = *reinterpret_cast<const floatx4*>(pb + (z0 + i) * step);
      }
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (z0 + i < ksplit) {
        a += t[i];
        b += u[i];
      }
  }
}

// h = silu(gate) * up, rounded to bf16 once, where the k range of the two projections was divided (an undivided one
// has this in its epilogue).  gate and up [ksplit][2 rows][f] fp32, partial, by choice; h [2 rows][f] bf16
__global__ __launch_bounds__(256) void gated_act_kernel(const float* gate, const float* up, int f, int ksplit, long long split_stride, uint16_t* h) {
  const int c = blockIdx.y * 256 + threadIdx.x;
  if (c >= f / 4) return;
  const long long at = (long long)blockIdx.x * f;
  floatx4 a, b;
  sum_two(gate + at + 4 * c, up + at + 4 * c, ksplit, split_stride, a, b);
  float o[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) o[i] = a[i] / (1.f + expf(-a[i])) * b[i];
  uint2 w;
  w.x = bf16_bits_rne(o[0]) | (bf16_bits_rne(o[1]) << 16);
  w.y = bf16_bits_rne(o[2]) | (bf16_bits_rne(o[3]) << 16);
  reinterpret_cast<uint2*>(h + at)[c] = w;
}

// f_top[r][k] = Expert_{idx[r][k]}(u_r) + u_r; f_mix[r] = sum_k s_k Expert_k(u_r) + u_r (Eq. 3).  y_parts [ksplit][rows][2][d] fp32: the chosen
// experts' (partial) outputs; u_rows [rows][d], f_top [rows][2][d], f_mix [rows][d] (or null) bf16
__global__ __launch_bounds__(256) void select_kernel(const float* y_parts, const uint16_t* u_rows, const float* s_top, int d, int ksplit, long long split_stride,
                                                     uint16_t* f_top, uint16_t* f_mix) {
  const int row = blockIdx.x;
  const int c = blockIdx.y * 256 + threadIdx.x;
  if (c >= d / 4) return;
  const uint2 uu = reinterpret_cast<const uint2*>(u_rows + (long long)row * d)[c];
  int lane_zero = 0;
  asm volatile("" : "+v"(lane_zero));  // (a vector load: the scalar one's trip was waited for in front of the results')
  const float s1 = s_top[2 * row + lane_zero], s2 = s_top[2 * row + 1 + lane_zero];
  const float* y = y_parts + (long long)(2 * row) * d + 4 * c;
  floatx4 a, b;
  if (ksplit == 1) {
    a = *reinterpret_cast<const floatx4*>(y);
    b = *reinterpret_cast<const floatx4*>(y + d);
  } else {
    sum_two(y, y + d, ksplit, split_stride, a, b);
  }
  const floatx4 u = {bf16_lo(uu.x), bf16_hi(uu.x), bf16_lo(uu.y), bf16_hi(uu.y)};
  auto store = [&](uint16_t* dst, const floatx4& v) {
    uint2 w;
    w.x = bf16_bits_rne(v[0]) | (bf16_bits_rne(v[1]) << 16);
    w.y = bf16_bits_rne(v[2]) | (bf16_bits_rne(v[3]) << 16);
    reinterpret_cast<uint2*>(dst)[c] = w;
  };
  store(f_top + ((long long)row * 2 + 0) * d, a + u);
  store(f_top + ((long long)row * 2 + 1) * d, b + u);
  if (f_mix) store(f_mix + (long long)row * d, s1 * a + s2 * b + u);
}

struct MoePlan {
  bool ring1, ring2;  // gate and up projections, output projection: in ring_gemm.hip
  int rows, used;     // `used` experts with at most so many rows each, as is likely
  int split1, split2;
  size_t g_off, up_off, h_off, y_off, total;
};
MoePlan moe_plan(int rows, int d, int f, int n) {
  MoePlan m;
  auto up = [](size_t v) { return (v + 255) / 256 * 256; };
  // the experts that rows choosing two of n each are likely to reach, and how many rows each of those has
  double missed = 1.0;
  for (int r = 0; r < rows; ++r) missed *= 1.0 - 2.0 / n;
  const int used = n * (1.0 - missed) < 2.0 ? 2 : (int)(n * (1.0 - missed) + 0.5);
  const int each = (2 * rows + used - 1) / used;
  const double mean = 2.0 * rows / n, likely = std::ceil(mean + 3.0 * std::sqrt(mean * (1.0 - 2.0 / n)));
  m.used = used;
  m.rows = likely < kRingRows ? (int)likely : kRingRows;
  const RingExperts x{mean, likely > kRingRows && mean > 28.0, used, n < 2 * rows ? n : 2 * rows};
  m.ring1 = ring_gemm_takes_pair(x, f, d);
  m.ring2 = ring_gemm_takes_down(x, d, f);
  m.split1 = m.ring1 ? 1 : stream_gemm_ksplit(each, f, d, used, true, 7000);  // gate and up in one launch
  m.split2 = m.ring2 ? 1 : stream_gemm_ksplit(each, d, f, used, false, 0);
  const size_t pre = m.split1 > 1 ? up((size_t)m.split1 * 2 * rows * f * 4) : 0;
  m.g_off = 0;
  m.up_off = pre;
  m.h_off = 2 * pre;
  m.y_off = m.h_off + up((size_t)2 * rows * f * 2);
  m.total = m.y_off + up((size_t)m.split2 * 2 * rows * d * 4);
  return m;
}


// ------------------------------------------------------------------ plain linear layer
// part [ksplit][m*n] fp32; residual (or null) and out_bf16 (or null) [m*n] bf16, out_f32 (or null) fp32
__global__ __launch_bounds__(256) void linear_finish_kernel(const float* part, const uint16_t* residual, long long n_out, int ksplit, float* out_f32,
                                                            uint16_t* out_bf16) {
  const long long i = ((long long)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i >= n_out) return;
  const bool vec = (n_out & 3) == 0 && (reinterpret_cast<size_t>(residual) & 7) == 0 && (reinterpret_cast<size_t>(out_bf16) & 7) == 0 &&
                   (reinterpret_cast<size_t>(out_f32) & 15) == 0;
  if (vec) {
    uint2 q = {0u, 0u};
    if (residual) q = *reinterpret_cast<const uint2*>(residual + i);
    floatx4 v = sum_parts(part + i, ksplit, n_out);
    if (residual) v += floatx4{bf16_lo(q.x), bf16_hi(q.x), bf16_lo(q.y), bf16_hi(q.y)};
    if (out_f32) *reinterpret_cast<floatx4*>(out_f32 + i) = v;
    if (out_bf16) {
      uint2 w;
      w.x = bf16_bits_rne(v[0]) | (bf16_bits_rne(v[1]) << 16);
      w.y = bf16_bits_rne(v[2]) | (bf16_bits_rne(v[3]) << 16);
      *reinterpret_cast<uint2*>(out_bf16 + i) = w;
    }
    return;
  }
  for (long long j = i; j < i + 4 && j < n_out; ++j) {
    float v = part[j];
    for (int z = 1; z < ksplit; ++z) v += part[j + z * n_out];
    if (residual) v += bf16_lo(residual[j]);
    if (out_f32) out_f32[j] = v;
    if (out_bf16) out_bf16[j] = (uint16_t)bf16_bits_rne(v);
  }
}

// parts of a product with few output columns, at most 64 MB of partial results
int capped_ksplit(int m, int n, int k, int split_ns, double* ns = nullptr) {
  int s = stream_gemm_ksplit(m, n, k, 1, false, split_ns, ns);
  while (s > 1 && (size_t)s * m * n * 4 > ((size_t)64 << 20)) --s;
  return s;
}

struct RowPlan {
  bool ring, stats;  // stats: the product leaves the rows' statistics (row_stats_kernel)
  int per_thread, parts, part_len, ksplit;
  size_t ms_off, key_off, part_off;
  size_t total, most;  // bytes that the call needs, and all that it has a use for
};

// `bytes`: of the workspace
RowPlan row_plan(int rows, int d_model, int vocab, size_t bytes) {
  RowPlan r;
  const size_t m = 2 * (size_t)rows;
  // Short parts spread a few rows over the CUs; with many rows long ones keep the grid at one turn of eight workgroups
  // per CU (20 rows of 128256, all kernels: 199 us in parts of 2048, 202 in parts of 1024, 200 in parts of 4096, and 209
  // in parts of 8192 with the top-k of a row in its first part's workgroup).
  r.per_thread = 4;
  while (r.per_thread < kPartPerThreadMax && (vocab + kPartThreads * r.per_thread - 1) / (kPartThreads * r.per_thread) * (long long)m > 8LL * device_cu_count())
    r.per_thread *= 2;
  r.parts = (vocab + kPartThreads * r.per_thread - 1) / (kPartThreads * r.per_thread);
  r.part_len = ((vocab + r.parts - 1) / r.parts + 3) / 4 * 4;
  auto up = [](size_t v) { return (v + 255) / 256 * 256; };
  r.ms_off = up(m * (size_t)d_model * 2);
  r.key_off = r.ms_off + up(m * r.parts * 2 * 4);
  r.part_off = r.key_off + up(m * r.parts * kMaxTopK * 8);
  r.ring = ring_gemm_takes_heads((int)m, vocab);
  r.ksplit = r.ring ? 1 : capped_ksplit((int)m, vocab, d_model, 0);
  r.total = r.part_off + (r.ksplit > 1 ? up((size_t)r.ksplit * m * vocab * 4) : 0);
  // The statistics come with the product wherever a workgroup has all of k and mixes its rows itself (launch_stream_gemm_heads).
  // Calls, us, in two launches over the rows (long rows) or one (short ones) / like this: 2 rows of 32000 x 4096 53.9 / 51.6, 20
  // of 128256 x 4096 189.5 / 186.9, 40 of 32000 x 4096 57.8 / 54.6, of 60000 x 1024 40.8 / 38.7, 64 of 128256 x 4096 221 / 218, 2 of 30000 x 512 16.7 /
  // 14.5; short rows, 64 of 32000 x 4096 61.7 / 61.3, of 20000 x 1024 22.6 / 22.3, 40 of 16384 x 4096 35.7 / 35.7.  The distributions' distance from
  // those in 64 bits of the same logits, mean of 480 - 768 rows: 0.94 - 0.995 times what it was in seven shapes at temperatures of 0.3 - 2.5.
  // They are more bytes than the parts of 4096 entries and their candidates where d_model is small; a workspace that holds those only still
  // serves the call, in the two launches.
  const size_t stat_bytes = up(m * ((vocab + kStatColumns - 1) / kStatColumns) * 8);
  const bool can = !r.ring && r.ksplit == 1 && m <= 64;
  r.stats = can && stat_bytes <= bytes;
  r.most = can && stat_bytes > r.total ? stat_bytes : r.total;
  return r;
}

}  // namespace

size_t draft_heads_workspace_bytes(int rows, int d_model, int vocab) { return row_plan(rows, d_model, vocab, 0).most; }
size_t draft_heads_least_bytes(int rows, int d_model, int vocab) { return row_plan(rows, d_model, vocab, 0).total; }

hipError_t launch_draft_heads(const DraftHeadsArgs& a, hipStream_t stream) {
  const int m = 2 * a.rows;
  const RowPlan rp = row_plan(a.rows, a.d_model, a.vocab, a.workspace_bytes);
  char* ws = static_cast<char*>(a.workspace);
  MixParams mp;
  mp.f_top = static_cast<const unsigned short*>(a.f_top);
  mp.s_top = a.s_top;
  mp.x = reinterpret_cast<unsigned short*>(ws);
  mp.rows = a.rows; mp.d = a.d_model; mp.mode = a.mode; mp.alpha = a.alpha; mp.beta = a.beta;
  const bool mixes = rp.ring || m <= 64;  // the product makes its rows itself (see launch_stream_gemm_heads)
  hipError_t e = hipSuccess;
  if (!mixes) {
    if ((e = launch_kernel(head_inputs_kernel, dim3((unsigned)(((long long)a.rows * (a.d_model / 8) + 63) / 64)), dim3(64), 0, stream, mp)) != hipSuccess) return e;
  }

  const uint16_t *x = mixes ? mp.f_top : reinterpret_cast<const uint16_t*>(ws), *w = static_cast<const uint16_t*>(a.w_head);
  float* parts = rp.ksplit > 1 ? reinterpret_cast<float*>(ws + rp.part_off) : nullptr;
  StreamGemmArgs g{};
  g.x = x; g.w = w; g.y = parts ? parts : a.logits;
  g.m = m; g.n = a.vocab; g.k = a.d_model;
  g.ksplit = rp.ksplit; g.y_split = (long long)m * a.vocab; g.batch = 1;
  g.s_top = a.s_top; g.heads_mode = a.mode; g.alpha = a.alpha; g.beta = a.beta;
  g.stats = rp.stats ? reinterpret_cast<float2*>(ws) : nullptr;  // (nothing else is in the workspace then)
  // (1 / T below the largest float has its log2(e)-fold beyond it from T = 4.24e-39 downwards: then the first part is the largest float, and
  // the second what is left, a number too.  An infinite one made rows none by zero times it.)
  const double scale = (double)(1.0f / a.temperature) * 1.4426950408889634;
  g.scale_hi = scale > (double)FLT_MAX ? FLT_MAX : (float)scale; g.scale_lo = (float)(scale - (double)g.scale_hi);
  e = rp.ring ? launch_ring_gemm_heads(g, stream) : mixes ? launch_stream_gemm_heads(g, stream) : launch_stream_gemm(g, stream);
  if (e != hipSuccess) return e;

  SoftParams sp;
  sp.logits = a.logits; sp.sums = parts; sp.ksplit = rp.ksplit; sp.probs = a.draft_probs; sp.tk_ids = a.topk_tokens; sp.tk_probs = a.topk_probs;
  sp.part_ms = reinterpret_cast<float*>(ws + rp.ms_off);
  sp.keys = reinterpret_cast<unsigned long long*>(ws + rp.key_off);
  sp.n_rows = m; sp.vocab = a.vocab; sp.k = a.top_k; sp.parts = rp.parts; sp.part_len = rp.part_len;
  sp.inv_temp = 1.0f / a.temperature;
  sp.stats = g.stats; sp.blocks = (a.vocab + kStatColumns - 1) / kStatColumns;
  sp.scale_hi = g.scale_hi; sp.scale_lo = g.scale_lo;
  if (!rp.stats && rows_whole(m, a.vocab)) {
    sp.parts = 1;
    sp.part_len = (a.vocab + 3) / 4 * 4;
    auto whole = [&](auto per_thread) {
      return launch_kernel(row_whole_kernel<decltype(per_thread)::value>, dim3((unsigned)m), dim3(kRowThreads), 0, stream, sp);
    };
    switch ((a.vocab + 4 * kRowThreads - 1) / (4 * kRowThreads)) {  // (four entries a thread more take 0.5 us: 4 tokens and 9000 entries in 12 instead of 16 13.8 / 13.3)
      case 1: return whole(std::integral_constant<int, 4>());
      case 2: return whole(std::integral_constant<int, 8>());
      case 3: return whole(std::integral_constant<int, 12>());
      case 4: return whole(std::integral_constant<int, 16>());
      case 5: return whole(std::integral_constant<int, 20>());
      case 6: return whole(std::integral_constant<int, 24>());
      case 7: return whole(std::integral_constant<int, 28>());
      default: return whole(std::integral_constant<int, 32>());
    }
  }
  switch (rp.per_thread) {
    case 4: return launch_rows<4>(sp, stream);
    case 8: return launch_rows<8>(sp, stream);
    default: return launch_rows<16>(sp, stream);
  }
}

size_t moe_experts_workspace_bytes(int rows, int d_model, int d_ff, int n_experts) {
  return moe_plan(rows, d_model, d_ff, n_experts).total;
}

hipError_t launch_moe_experts(const MoeArgs& a, hipStream_t stream) {
  const MoePlan mp = moe_plan(a.rows, a.d_model, a.d_ff, a.n_experts);
  char* ws = static_cast<char*>(a.workspace);
  hipError_t e;
  const uint16_t* u = static_cast<const uint16_t*>(a.u);
  if ((e = launch_kernel(router_kernel, dim3(a.rows), dim3(256), 0, stream, u, static_cast<const uint16_t*>(a.centroids), a.d_model, a.n_experts, a.s_top,
                     a.expert_idx)) != hipSuccess) return e;

  // Each expert runs for the rows that chose it only
  uint16_t* h = reinterpret_cast<uint16_t*>(ws + mp.h_off);
  StreamGemmArgs g{};
  g.x = u; g.m = a.rows; g.n = a.d_ff; g.k = a.d_model;
  g.batch = a.n_experts; g.w_batch = (long long)a.d_ff * a.d_model;
  g.sel = a.expert_idx;
  g.ksplit = mp.split1; g.y_split = (long long)a.rows * 2 * a.d_ff;
  g.w = static_cast<const uint16_t*>(a.w_gate); g.w2 = static_cast<const uint16_t*>(a.w_up);
  if (mp.split1 > 1) {
    g.y = reinterpret_cast<float*>(ws + mp.g_off); g.y2 = reinterpret_cast<float*>(ws + mp.up_off);
  } else {
    g.act = h;
  }
  if ((e = mp.ring1 ? launch_ring_gemm_pair(g, mp.rows, mp.used, stream) : launch_stream_gemm_pair(g, stream)) != hipSuccess) return e;  // gate and up projections of all experts
  if (mp.split1 > 1) {
    if ((e = launch_kernel(gated_act_kernel, dim3(2 * a.rows, (unsigned)((a.d_ff / 4 + 255) / 256)), dim3(256), 0, stream, g.y, g.y2, a.d_ff, mp.split1,
                       g.y_split, h)) != hipSuccess) return e;
  }
  StreamGemmArgs o{};
  o.x = h; o.m = a.rows; o.n = a.d_model; o.k = a.d_ff;
  o.batch = a.n_experts; o.w_batch = (long long)a.d_model * a.d_ff;
  o.sel = a.expert_idx;
  o.ksplit = mp.split2; o.y_split = (long long)a.rows * 2 * a.d_model;
  o.w = static_cast<const uint16_t*>(a.w_down); o.y = reinterpret_cast<float*>(ws + mp.y_off);
  if ((e = mp.ring2 ? launch_ring_gemm_down(o, mp.rows, mp.used, stream) : launch_stream_gemm_down(o, stream)) != hipSuccess) return e;

  return launch_kernel(select_kernel, dim3(a.rows, (unsigned)((a.d_model / 4 + 255) / 256)), dim3(256), 0, stream, o.y, u, a.s_top, a.d_model, mp.split2,
                     o.y_split, static_cast<uint16_t*>(a.f_top), static_cast<uint16_t*>(a.f_mix));
}

namespace {
constexpr int kLinearSplitNs = 3500;  // linear_finish_kernel

// Either narrow_gemm_kernel (narrow.parts > 0) or stream_gemm_kernel with ksplit parts of k
struct LinearPlan {
  NarrowPlan narrow;
  int ksplit;
};
LinearPlan plan_linear(int m, int n, int k) {
  LinearPlan p{narrow_plan(m, n, k), 1};
  const int forced = tuning().narrow_gemm;
  if (forced > 0 && p.narrow.parts > 0) return p;
  if (forced < 0 && m <= 64 && p.narrow.parts > 0 && 2 * p.narrow.strips * p.narrow.blocks * p.narrow.parts > device_cu_count()) return p;
  // (few columns leave CUs without a strip; the estimate of the other way comes out 10 % low, more so for many rows.  Of 100 shapes
  // with 65 - 128 rows none that is taken here is slower, 0.99 - 2.6 times as fast; beyond the line, k very long beside the
  // number of columns: 128 x 4096 x 16384 46 against 57 us, 80 x 5120 x 10240 32 against 36.)
  double ns = 0.0;
  p.ksplit = capped_ksplit(m, n, k, kLinearSplitNs, &ns);
  if (forced == 0 || p.narrow.ns >= (m <= 64 ? 1.04 : 1.06) * ns) p.narrow.parts = 0;
  return p;
}
// A call asks for its plan three times (its bytes, their check, the launch), 0.1 - 1 us each of a thread that has 6 us for a small
// layer: a thread keeps its last answer.  (A layer of 1024 columns for 10 rows, bound by its enqueueing: 24.0 us a pass, 23.7 like this.)
LinearPlan linear_plan(int m, int n, int k) {
  struct Last {
    int m, n, k, cus, forced;
    LinearPlan plan;
  };
  static thread_local Last last{};
  const int cus = device_cu_count(), forced = tuning().narrow_gemm;
  if (last.m != m || last.n != n || last.k != k || last.cus != cus || last.forced != forced) last = Last{m, n, k, cus, forced, plan_linear(m, n, k)};
  return last.plan;
}
}  // namespace

namespace {
size_t linear_writes(const LinearPlan& p, int m, int n) {  // bytes
  return p.narrow.parts > 0 ? narrow_gemm_bytes(p.narrow) : p.ksplit > 1 ? (size_t)p.ksplit * m * n * 4 : 0;
}
}  // namespace
bool linear_call_writes(int m, int n, int k) { return linear_writes(linear_plan(m, n, k), m, n) > 0; }

size_t linear_workspace_bytes(int m, int n, int k) {
  const size_t need = linear_writes(linear_plan(m, n, k), m, n);
  return need < 256 ? 256 : (need + 255) / 256 * 256;
}

hipError_t launch_linear(const LinearArgs& a, hipStream_t stream) {
  const LinearPlan lp = linear_plan(a.m, a.n, a.k);
  StreamGemmArgs g{};
  g.x = static_cast<const uint16_t*>(a.x); g.w = static_cast<const uint16_t*>(a.w);
  g.m = a.m; g.n = a.n; g.k = a.k; g.ksplit = lp.ksplit; g.y_split = (long long)a.m * a.n; g.batch = 1;
  if (lp.narrow.parts > 0 || lp.ksplit == 1) {
    g.finish = true;
    g.y = a.out_f32; g.residual = static_cast<const uint16_t*>(a.residual); g.out_bf16 = static_cast<uint16_t*>(a.out_bf16);
    return lp.narrow.parts > 0 ? launch_narrow_gemm(g, lp.narrow, a.workspace, stream) : launch_stream_gemm(g, stream);
  }
  g.y = static_cast<float*>(a.workspace);
  hipError_t e = launch_stream_gemm(g, stream);
  if (e != hipSuccess) return e;
  const long long n_out = (long long)a.m * a.n;
  return launch_kernel(linear_finish_kernel, dim3((unsigned)((n_out + 1023) / 1024)), dim3(256), 0, stream, g.y, static_cast<const uint16_t*>(a.residual),
                     n_out, lp.ksplit, a.out_f32, static_cast<uint16_t*>(a.out_bf16));
}

}  // namespace jk
