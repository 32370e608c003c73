// Tree-masked verification attention, fp32 inputs.
//
// Same definition as the bf16 kernel (Section 2.1 step 2; Section 3.1.2 tree mask), fp32 end to end for accuracy-critical
// shapes.  One workgroup per (sequence, KV head, 16 query rows, key split); its waves take blocks of 16 keys in turn, keep
// a running maximum and sum per row, and meet once at the end, in LDS.
//
// What bounds it: for small calls the instructions of a lone wave (5 - 8 cycles each; a block of 16 keys takes 2400 cycles with
// its operands there) and the trips to memory in front of them.  So a wave has a block's K and V in flight at once and the next
// block's K behind them, the prefix's and the tree's alike; who has a block of the tree makes the ancestors of its rows while the
// keys come; at the end a wave scales its own sums, and what is left to do for the result is adding.  For large calls the
// products bind, which run on v_mfma_f32_16x16x4_f32 (full fp32) with K and V straight from L2 in operand layout, each read once
// for 16 rows.  S^T = K Q^T leaves a lane with four keys of one row: exactly what the second product, O^T = V^T P^T, takes as its
// operand, so the weights never leave their registers.  An undivided key range needs no second launch.
//
// A small head's first block is asked for before the prefix length is known, K and V, where the key range is undivided; with more
// than 64 columns it is not, and not in front of the ancestors either: what a CU draws (some 60 bytes per ns, 200 KB for eight
// waves' rows, K and V of 128 columns) takes longer than the trip that it saves, and the exchanges between lanes wait among it (3 -
// 10 % more for trees of 64 nodes).  4 heads of 64, 10 nodes and 138 keys: 16.9 us with one workgroup per query row and a thread
// per key and column (the second launch included), 7.9 with the tree's ancestors made by one wave for all, 6.2 with the first
// block's K alone asked for early, 5.8 like this (6.7 with sixteen waves, of which none has two blocks); 45 drawn and edge calls of
// all head dimensions 1.025 times as fast as with the K of a divided range's first part and of larger heads asked for early too
// (0.975 - 1.10); 4 sequences, 8 heads of 128, 52 nodes, 2100 keys 481, 56.4 and 56.
#include <type_traits>

#include "jk_ancestors.h"
#include "jk_device.h"
#include "jk_divide.h"
#include "jk_wave.h"

namespace jk {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

struct FParams {
  const float *q, *kc, *vc, *kt, *vt;
  const int32_t *parent, *prefix_len;
  float* part_o;
  float2* part_ml;
  float* out;     // undivided key range: the result
  unsigned* err;  // the workspace's sticky device error word
  unsigned* words;  // divided range, merged by the last of a row tile's workgroups: a word each (f32_word); or null
  int B, T, Hkv, G, M, m_pad, D, max_prefix, splits, over_hkv;
  long long q_sb, q_st, q_sh, kc_sb, kc_sl, kc_sh, kt_sb, kt_st, kt_sh, o_sb, o_st, o_sh;
  unsigned long long mg_g, mg_hkv;  // for n / G and n / Hkv, with over_g and over_hkv (jk_divide.h)
  int over_g;
  float scale;
};
static_assert(sizeof(FParams) > 192 && sizeof(FParams) <= 256, "four lines of kernel arguments");

// KJ: 16-column chunks of a head (rounded up); WAVES: by how many registers that leaves.  WHOLE: an undivided key range of a
// small head, whose first loads do not wait for the prefix length
template <int KJ>
constexpr int waves_for() { return KJ <= 8 ? 8 : 4; }

template <int KJ, int WAVES, bool WHOLE>
__global__ __launch_bounds__(64 * WAVES, KJ <= 8 ? (WAVES + 3) / 4 : 1) void tva_f32_kernel(FParams p) {
  constexpr int DB = (KJ + 3) / 4, LDO = 64 * DB + 4;
  __shared__ float tops[WAVES][16];     // a wave's maximum of a row,
  __shared__ float2 shares[WAVES][16];  // and its share of the row's sum, beside the maximum of all
  extern __shared__ __attribute__((aligned(16))) float osum[];  // [WAVES][16][LDO]

  {  // every 64-byte line of the kernel arguments at once: the compiler fetches them in several dependent batches
    typedef __attribute__((address_space(4))) const unsigned kernarg_word;
    kernarg_word* ka = (kernarg_word*)__builtin_amdgcn_kernarg_segment_ptr();
    const unsigned a0 = ka[0], a1 = ka[16], a2 = ka[32], a3 = ka[48];
    asm volatile("" ::"s"(a0), "s"(a1), "s"(a2), "s"(a3));
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int c = lane & 15, g = lane >> 4;
  const int split = blockIdx.x, row0 = blockIdx.y * 16;
  const int b = quotient((int)blockIdx.z, p.mg_hkv, p.over_hkv), kv = blockIdx.z - b * p.Hkv;
  const int D = p.D;
  const float* kc = p.kc + b * p.kc_sb + (long long)kv * p.kc_sh;
  const float* vc = p.vc + b * p.kc_sb + (long long)kv * p.kc_sh;
  const float* kt = p.kt + b * p.kt_sb + (long long)kv * p.kt_sh;
  const float* vt = p.vt + b * p.kt_sb + (long long)kv * p.kt_sh;

  int lane_zero = 0;
  asm volatile("" : "+v"(lane_zero));  // (a vector load: a scalar one would be waited for with the arguments)
  const int L_raw = __hip_atomic_load(p.prefix_len + b + lane_zero, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int pa0 = p.parent[(long long)b * p.T + min(lane, p.T - 1)], pa1 = p.parent[(long long)b * p.T + min(lane + 64, p.T - 1)];
  const int m = min(row0 + c, p.M - 1), node = quotient(m, p.mg_g, p.over_g);  // this lane's query row (rows past the end repeat the last one)
  floatx4 q[KJ], k[KJ], v[DB][4];  // the row, and a block's K and V
  // column 16 j + 4 g of a row; columns past the end: the row's first ones, against zeros of q
  auto col = [&](int j) { return 16 * j + 4 * g < D ? 16 * j + 4 * g : 0; };

  // ---- this wave's blocks of 16 keys: of the tree's first, first + WAVES, ..., then of the prefix's wave, wave + WAVES, ...  The
  // tree's begin with the waves that have fewer of the prefix, if its length is the host's bound: so which wave has them, and
  // what it asks for first, does not depend on the length.  (At most 512 ranges of at most 65 664 keys.)
  const bool whole = WHOLE || p.splits == 1;
  int p_end, tree_begin, tree_end, n_mine_t, n_mine, first, k_begin;
  auto set_range = [&](int L, bool bound) {
    const int ktot = L + p.T;
    k_begin = whole ? 0 : (int)((unsigned)split * (unsigned)ktot / (unsigned)p.splits);
    const int k_end = whole ? ktot : (int)((unsigned)(split + 1) * (unsigned)ktot / (unsigned)p.splits);
    p_end = min(k_end, L);
    tree_begin = max(k_begin, L) - L;
    tree_end = k_end - L;
    const int n_prefix = max(p_end - k_begin + 15, 0) >> 4, n_tree = max(tree_end - tree_begin + 15, 0) >> 4;
    if (bound) first = (wave - n_prefix) & (WAVES - 1);
    n_mine_t = max(n_tree - first + WAVES - 1, 0) / (unsigned)WAVES;
    n_mine = n_mine_t + max(n_prefix - wave + WAVES - 1, 0) / (unsigned)WAVES;
  };
  struct Block {
    const float *k, *v;   // the rows
    long long stride;
    int key0, last;       // the first of them, and the last that counts
    bool tree;
  };
  auto block_at = [&](int i) {
    Block x;
    x.tree = i < n_mine_t;
    x.k = x.tree ? kt : kc;
    x.v = x.tree ? vt : vc;
    x.stride = x.tree ? p.kt_st : p.kc_sl;
    x.key0 = x.tree ? tree_begin + 16 * (first + WAVES * i) : k_begin + 16 * (wave + WAVES * (i - n_mine_t));
    x.last = (x.tree ? tree_end : p_end) - 1;
    return x;
  };
  auto load_k = [&](const Block& x, int c, int g) {
    const float* row = x.k + (long long)min(x.key0 + c, x.last) * x.stride;
#pragma unroll
    for (int j = 0; j < KJ; ++j) k[j] = *reinterpret_cast<const floatx4*>(row + (16 * j + 4 * g < D ? 16 * j + 4 * g : 0));
  };
  auto load_v = [&](const Block& x, int c, int g) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float* row = x.v + (long long)min(x.key0 + 4 * g + i, x.last) * x.stride;
#pragma unroll
      for (int d = 0; d < DB; ++d) v[d][i] = *reinterpret_cast<const floatx4*>(row + (64 * d + 4 * c < D ? 64 * d + 4 * c : 0));
    }
  };
  auto load_row = [&]() {
    const float* src = p.q + b * p.q_sb + node * p.q_st + (long long)(kv * p.G + m - node * p.G) * p.q_sh;
#pragma unroll
    for (int j = 0; j < KJ; ++j) q[j] = *reinterpret_cast<const floatx4*>(src + col(j));
  };
  auto length = [&]() {
    const int len = __builtin_amdgcn_readfirstlane(L_raw);
    return len < 0 ? 0 : (len > p.max_prefix ? p.max_prefix : len);
  };
  Block cur;
  load_row();
  if constexpr (WHOLE) {
    // The first block on the assumption that the length is the host's bound: one trip to memory for all of it.  (In a branch,
    // the compiler would wait for all of it where it waits for the length: a wave without a block asks for one key of the tree
    // in every lane.)
    set_range(p.max_prefix, true);
    const bool some = n_mine > 0;
    cur = block_at(0);
    if (!some) cur = Block{kt, vt, 0, 0, 0, true};
    load_k(cur, some ? c : 0, some ? g : 0);
    load_v(cur, some ? c : 0, some ? g : 0);
    set_range(length(), false);
    if (!cur.tree) cur.last = p_end - 1;
  } else {
    set_range(length(), true);
    cur = block_at(0);
  }
  dev::Ancestors seen{0ull, 0ull};
  if (n_mine_t > 0 || (split == 0 && wave == 0))
    seen = dev::ancestors_of(p.T, p.err, lane < p.T ? pa0 : -1, lane + 64 < p.T ? pa1 : -1, node, split == 0 && row0 == 0 && kv == 0 && wave == 0);
  if (!WHOLE && n_mine > 0) {
    load_k(cur, c, g);
    load_v(cur, c, g);
  }
  if (16 * KJ != D) {
#pragma unroll
    for (int j = 0; j < KJ; ++j)
      if (16 * j + 4 * g >= D) q[j] = floatx4{0.f, 0.f, 0.f, 0.f};
  }

  // A weight of zero - an unseen key's above all - leaves its value out, whatever that is.  The matrix product has one
  // value for sixteen rows' weights, so an infinity or a NaN reaches them all; it stays in the accumulators to the end, and
  // a wave that finds one there takes its keys once more, key by key.  (Looked for in the values themselves, in front of
  // each product: 57.0 us for 4 sequences, 8 heads of 128, 52 nodes, 2100 keys became 59.8.)
  floatx4 o[DB][4];
  float mx, sum;
  auto pass = [&](auto careful) {
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
      for (int i = 0; i < 4; ++i) o[d][i] = floatx4{0.f, 0.f, 0.f, 0.f};
    mx = -INFINITY;
    sum = 0.f;
    if (careful && n_mine > 0) {
      cur = block_at(0);
      load_k(cur, c, g);
    }
    for (int blk = 0; blk < n_mine; ++blk) {  // (its K and V have been asked for)
      const Block now = cur;
      if (16 * KJ != D) {  // (uniform; what stands in for columns past the end of a key with an infinity must not meet q's zeros)
#pragma unroll
        for (int j = 0; j < KJ; ++j)
          if (16 * j + 4 * g >= D) k[j] = floatx4{0.f, 0.f, 0.f, 0.f};
      }
      floatx4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < KJ; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) s = __builtin_amdgcn_mfma_f32_16x16x4f32(k[j][i], q[j][i], s, 0, 0, 0);
      if (blk + 1 < n_mine) {
        cur = block_at(blk + 1);
        load_k(cur, c, g);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) s[i] *= p.scale;
      if (now.tree || now.key0 + 15 > now.last) {  // (uniform) the keys that this lane's row sees, a bit each; then its four
        unsigned mine = ~0u;
        if (now.tree) mine = (unsigned)(now.key0 >= 64 ? seen.hi >> (now.key0 - 64) : now.key0 > 0 ? seen.lo >> now.key0 | seen.hi << (64 - now.key0) : seen.lo);
        mine &= (2u << min(now.last - now.key0, 15)) - 1u;
        mine >>= 4 * g;
#pragma unroll
        for (int i = 0; i < 4; ++i) s[i] = (mine >> i) & 1u ? s[i] : -INFINITY;
      }
      float top = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
      top = fmaxf(top, __uint_as_float(dev::other16(__float_as_uint(top), lane & 16)));
      top = fmaxf(top, __uint_as_float(dev::other32(__float_as_uint(top), lane & 32)));
      const float mn = fmaxf(mx, top), base = mn == -INFINITY ? 0.f : mn;
      if (__any(mn > mx && mx > -INFINITY)) {  // (nothing to rescale before the row's first key)
        const float f = expf(mx - base);
        sum *= f;
#pragma unroll
        for (int d = 0; d < DB; ++d)
#pragma unroll
          for (int i = 0; i < 4; ++i) o[d][i] *= f;
      }
      mx = mn;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        s[i] = expf(s[i] - base);
        sum += s[i];
      }
      if (careful) {
#pragma unroll 1
        for (int key = 0; key < 16; ++key) {
          const float mine = (key & 2) ? ((key & 1) ? s[3] : s[2]) : ((key & 1) ? s[1] : s[0]);
          const float w = __shfl(mine, 16 * (key >> 2) + c);
          const float* row = now.v + (long long)min(now.key0 + key, now.last) * now.stride;
#pragma unroll
          for (int d = 0; d < DB; ++d)
#pragma unroll
            for (int r = 0; r < 4; ++r) {  // (as everywhere: columns past the end take the row's first ones, and are not stored)
              const int at = 64 * d + 16 * g + 4 * r;
              const floatx4 x = *reinterpret_cast<const floatx4*>(row + (at < D ? at : 0));
#pragma unroll
              for (int e = 0; e < 4; ++e) o[d][e][r] = w != 0.f ? fmaf(x[e], w, o[d][e][r]) : o[d][e][r];
            }
        }
        continue;
      }
      if (now.key0 + 15 > now.last) {  // (a first block asked for beyond the prefix's end: what is there is nobody's value)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int d = 0; d < DB; ++d) v[d][i] = now.key0 + 4 * g + i > now.last ? floatx4{0.f, 0.f, 0.f, 0.f} : v[d][i];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int d = 0; d < DB; ++d)
#pragma unroll
          for (int e = 0; e < 4; ++e) o[d][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[d][i][e], s[i], o[d][e], 0, 0, 0);
      if (blk + 1 < n_mine) load_v(cur, c, g);
    }
  };
  pass(std::false_type());
  float wild = 0.f;
#pragma unroll
  for (int d = 0; d < DB; ++d)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) wild = fmaf(o[d][i][e], 0.f, wild);
  if (__any(wild != 0.f)) {
    asm volatile("" : "+v"(c), "+v"(g));  // (addresses are worked out afresh, not kept for this)
    pass(std::true_type());
  }

  // ---- the waves' shares of a row meet (each scaled by its own wave: worked out per column of the result, eight exponentials in
  // every thread, 7.9 us became 7.2 for the tiny call)
  sum += __uint_as_float(dev::other16(__float_as_uint(sum), lane & 16));
  sum += __uint_as_float(dev::other32(__float_as_uint(sum), lane & 32));
  if (g == 0) tops[wave][c] = mx;
  // (where this thread's columns of the result go, worked out while the others come)
  const int d4 = D / 4;
  int r = tid / d4, x = tid - r * d4;
  __syncthreads();
  float all = -INFINITY;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) all = fmaxf(all, tops[w][c]);
  const float f = mx == -INFINITY ? 0.f : expf(mx - all);
  if (g == 0) shares[wave][c] = make_float2(sum * f, all);
  float* mine = osum + (wave * 16 + c) * LDO + 16 * g;  // (a lane has 16 columns of its row in each 64)
#pragma unroll
  for (int d = 0; d < DB; ++d)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      *reinterpret_cast<floatx4*>(mine + 64 * d + 4 * r) = floatx4{o[d][0][r] * f, o[d][1][r] * f, o[d][2][r] * f, o[d][3][r] * f};
  __syncthreads();
  for (int i = tid; i < 16 * d4; i += 64 * WAVES) {
    if (i != tid) {
      r = i / d4;
      x = i - r * d4;
    }
    const int row = row0 + r;
    if (row >= p.M) break;
    floatx4 t = {0.f, 0.f, 0.f, 0.f};
    float tot = 0.f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      t += *reinterpret_cast<const floatx4*>(osum + (w * 16 + r) * LDO + 4 * x);
      tot += shares[w][r].x;
    }
    if (p.splits == 1) {
      const int n = quotient(row, p.mg_g, p.over_g);
      float* dst = p.out + b * p.o_sb + n * p.o_st + (long long)(kv * p.G + row - n * p.G) * p.o_sh;
      const float inv = 1.f / tot;  // (tot > 0: every row sees at least its own tree key)
      *reinterpret_cast<floatx4*>(dst + 4 * x) = floatx4{t[0] * inv, t[1] * inv, t[2] * inv, t[3] * inv};
    } else {
      const long long prow = ((long long)(b * p.Hkv + kv) * p.splits + split) * p.m_pad + row;
      const float2 ml = make_float2(shares[0][r].y, tot);
      if (p.words) {
        dev::store_through(p.part_o + prow * D + 4 * x, __builtin_bit_cast(dev::store_u32x4, t));
        if (x == 0) dev::store_through(p.part_ml + prow, __builtin_bit_cast(dev::store_u32x2, ml));
      } else {
        *reinterpret_cast<floatx4*>(p.part_o + prow * D + 4 * x) = t;
        if (x == 0) p.part_ml[prow] = ml;
      }
    }
  }
  if constexpr (!WHOLE) {
    if (p.splits == 1 || !p.words) return;
    // ---- Merge of the parts by the last of the row tile's workgroups to come: nobody waits, and the sum is the same whoever it is.
    // Results go through to memory in front of the count and are read past the caches (the workgroups run on different XCDs).
    // With a second launch for it before, a call: two sequences, 16 heads of 64, 3 nodes, 1811 keys in front 9.7 / 9.0 us; 4 of 80, 2 nodes,
    // 581 keys 9.7 / 8.5; 2 of 64, 3 nodes, 705 keys 8.6 / 7.3.
    __shared__ int last_s;
    dev::wait_vm<0>();
    __syncthreads();
    if (tid == 0) {
      unsigned* word = p.words + f32_word(blockIdx.z * gridDim.y + blockIdx.y);
      const bool last = __hip_atomic_fetch_add(word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)p.splits - 1u;
      if (last) __hip_atomic_store(word, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      last_s = last;
    }
    __syncthreads();
    if (!__builtin_amdgcn_readfirstlane(last_s)) return;
    const long long first = (long long)(b * p.Hkv + kv) * p.splits * p.m_pad + row0;  // the first part's first row
    const uint64_t* pairs = reinterpret_cast<const uint64_t*>(p.part_ml) + first;
    // (a unit's parts are below 2^31 bytes by the host's choice)
    const auto sums = __builtin_amdgcn_make_buffer_rsrc(p.part_o + first * D, 0, ((p.splits - 1) * p.m_pad + min(16, p.M - row0)) * D * 4, 0x00020000);
    // 4 * WAVES threads a row, each all of its columns at once: with one after the other, of 256, a trip to memory each
    // (8 sequences, 4 heads, 10 nodes, 138 keys 16.6 us / 14.1 so)
    constexpr int LANES = 4 * WAVES, COLS = (4 * KJ + LANES - 1) / LANES;
    const int r = tid / LANES, x = tid % LANES, row = row0 + r;
    if (row >= p.M) return;
    auto merge = [&](auto at_once) {  // (as many parts under way as there are, and no more: 8 for three of them took as long again)
      constexpr int AT_ONCE = decltype(at_once)::value;
      floatx4 t[COLS];
#pragma unroll
      for (int c = 0; c < COLS; ++c) t[c] = floatx4{0.f, 0.f, 0.f, 0.f};
      float tot = 0.f, top = -INFINITY;
      for (int s0 = 0; s0 < p.splits; s0 += AT_ONCE) {
        uint64_t ml[AT_ONCE];
        u32x4 o4[AT_ONCE][COLS];
#pragma unroll
        for (int u = 0; u < AT_ONCE; ++u) ml[u] = __hip_atomic_load(pairs + (long long)min(s0 + u, p.splits - 1) * p.m_pad + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int u = 0; u < AT_ONCE; ++u)
#pragma unroll
          for (int c = 0; c < COLS; ++c)
            o4[u][c] = __builtin_amdgcn_raw_buffer_load_b128(sums, ((min(s0 + u, p.splits - 1) * p.m_pad + r) * D + 4 * min(x + LANES * c, d4 - 1)) * 4, 0, dev::kDeviceScope);
        float here = top;
        float part_top[AT_ONCE], part_sum[AT_ONCE];
#pragma unroll
        for (int u = 0; u < AT_ONCE; ++u) {  // (a part without a key that the row sees, and what stands in for one past the last: no weight)
          part_sum[u] = s0 + u < p.splits ? __uint_as_float((unsigned)(ml[u] >> 32)) : 0.f;
          part_top[u] = dev::part_top(__uint_as_float((unsigned)ml[u]), part_sum[u]);
          here = fmaxf(here, part_top[u]);
        }
        const float base = here == -INFINITY ? 0.f : here, f = expf(top - base);  // (0 in front of the first)
        tot *= f;
#pragma unroll
        for (int c = 0; c < COLS; ++c) t[c] *= f;
        top = here;
#pragma unroll
        for (int u = 0; u < AT_ONCE; ++u) {
          const float w = expf(part_top[u] - base);
          tot = fmaf(part_sum[u], w, tot);
          if (w != 0.f) {
#pragma unroll
            for (int c = 0; c < COLS; ++c) {
              const floatx4 own = __builtin_bit_cast(floatx4, o4[u][c]);
#pragma unroll
              for (int e = 0; e < 4; ++e) t[c][e] = fmaf(own[e], w, t[c][e]);
            }
          }
        }
      }
      const int n = quotient(row, p.mg_g, p.over_g);
      float* dst = p.out + b * p.o_sb + n * p.o_st + (long long)(kv * p.G + row - n * p.G) * p.o_sh;
      const float inv = 1.f / tot;
#pragma unroll
      for (int c = 0; c < COLS; ++c)
        if (x + LANES * c < d4) *reinterpret_cast<floatx4*>(dst + 4 * (x + LANES * c)) = floatx4{t[c][0] * inv, t[c][1] * inv, t[c][2] * inv, t[c][3] * inv};
    };
    if (p.splits <= 4) merge(std::integral_constant<int, 4>());
    else if (p.splits <= 8 || KJ > 5) merge(std::integral_constant<int, 8>());
    else merge(std::integral_constant<int, 16>());
  }
}

template <int KJ, int WAVES, bool WHOLE>
hipError_t launch_waves(const FParams& fp, hipStream_t stream) {
  constexpr int SMEM = WAVES * 16 * (64 * ((KJ + 3) / 4) + 4) * 4;
  static LdsLimitRaised raised;
  if (hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(tva_f32_kernel<KJ, WAVES, WHOLE>), SMEM, raised); e != hipSuccess) return e;
  return launch_kernel(tva_f32_kernel<KJ, WAVES, WHOLE>, dim3(fp.splits, (fp.M + 15) / 16, fp.B * fp.Hkv), dim3(64 * WAVES), SMEM, stream, fp);
}
template <int KJ>
hipError_t launch_kj(const FParams& fp, hipStream_t stream) {
  if constexpr (KJ == 4) {
    if (fp.splits == 1) return launch_waves<4, 8, true>(fp, stream);
  }
  return launch_waves<KJ, waves_for<KJ>(), false>(fp, stream);
}

}  // namespace

// Up to 16 parts, 8 for four waves (the last workgroup of a row tile reads them all: beyond that the merging launch, which spreads
// them over the CUs; head_dim 256, 16 parts 25.4 us in the kernel, 24.2 with the launch, 64 6.5 % to the kernel), with a word for each row tile
bool f32_merges(const jk_attn_desc& d, const AttnPlan& pl) {
  const int most_parts = d.head_dim > 128 ? 8 : 16;
  const long long tiles = (long long)d.batch * d.n_kv_heads * ((pl.m_rows + 15) / 16);
  return pl.parts > 1 && pl.parts <= most_parts && tiles <= kMaxCounted && tuning().attn_fused != 0 &&
         (long long)pl.parts * pl.m_pad * d.head_dim * 4 < (1LL << 31);
}

hipError_t launch_tva_f32(const AttnArgs& a, const AttnPlan& pl, hipStream_t stream) {
  FParams fp;
  fp.q = static_cast<const float*>(a.q);
  fp.kc = static_cast<const float*>(a.k_cache);
  fp.vc = static_cast<const float*>(a.v_cache);
  fp.kt = static_cast<const float*>(a.k_tree);
  fp.vt = static_cast<const float*>(a.v_tree);
  fp.parent = a.parent;
  fp.prefix_len = a.prefix_len;
  fp.part_o = a.part_o;
  fp.part_ml = a.part_ml;
  fp.err = a.err;
  fp.words = a.sync;
  const jk_attn_desc& d = a.d;
  fp.B = d.batch; fp.T = d.n_tree; fp.Hkv = d.n_kv_heads; fp.G = d.n_q_heads / d.n_kv_heads;
  fp.M = pl.m_rows; fp.m_pad = pl.m_pad; fp.D = d.head_dim; fp.max_prefix = a.max_prefix_len;
  fp.splits = pl.parts;
  fp.q_sb = d.q_stride_b; fp.q_st = d.q_stride_t; fp.q_sh = d.q_stride_h;
  fp.kc_sb = d.kc_stride_b; fp.kc_sl = d.kc_stride_l; fp.kc_sh = d.kc_stride_h;
  fp.kt_sb = d.kt_stride_b; fp.kt_st = d.kt_stride_t; fp.kt_sh = d.kt_stride_h;
  fp.out = static_cast<float*>(a.out);
  fp.o_sb = d.o_stride_b; fp.o_st = d.o_stride_t; fp.o_sh = d.o_stride_h;
  const Divisor by_g = divisor(fp.M, fp.G), by_hkv = divisor((long long)fp.B * fp.Hkv, fp.Hkv);
  fp.mg_g = by_g.mg; fp.over_g = by_g.over;
  fp.mg_hkv = by_hkv.mg; fp.over_hkv = by_hkv.over;
  fp.scale = a.scale_log2;  // for this path the host passes the plain softmax scale here
  switch ((d.head_dim + 15) / 16) {
    case 1: case 2: case 3:
    case 4: return launch_kj<4>(fp, stream);
    case 5: return launch_kj<5>(fp, stream);
    case 6: return launch_kj<6>(fp, stream);
    case 7:
    case 8: return launch_kj<8>(fp, stream);
    default: return launch_kj<16>(fp, stream);
  }
}

}  // namespace jk
