// Tree-masked verification attention, fp32 inputs.
//
// Same definition as the bf16 kernel (Section 2.1 step 2; Section 3.1.2 tree mask), fp32 end to end for accuracy-critical
// shapes.  One workgroup per (sequence, KV head, 16 query rows, key split); its waves take blocks of 16 keys in turn, keep
// a running maximum and sum per row, and meet once at the end, in LDS.
//
// What bounds it: for small calls the instructions of a lone wave (5 - 8 cycles each; a block of 16 keys takes 2400 cycles with
// its operands there) and the trips to memory in front of them.  So a wave has a block's K and V in flight at once and the next
// block's K behind them, the prefix's and the tree's alike, and asks for the first block's K before the prefix length is known;
// who has a block of the tree makes the ancestors of its rows while the keys come; at the end a wave scales its own sums, and
// what is left to do for the result is adding.  For large calls the products bind, which run on v_mfma_f32_16x16x4_f32 (full
// fp32) with K and V straight from L2 in operand layout, each read once for 16 rows.  S^T = K Q^T leaves a lane with four keys
// of one row: exactly what the second product, O^T = V^T P^T, takes as its operand, so the weights never leave their registers.
// An undivided key range needs no second launch.  4 heads of 64, 10 nodes and 138 keys: 16.9 us with one workgroup per query
// row and a thread per key and column (the second launch included), 7.9 with the tree's ancestors made by one wave for all, its
// keys asked for behind a barrier and the waves' weights worked out by every thread of the result, 6.2 like this; 4 sequences, 8
// heads of 128, 52 nodes, 2100 keys 481, 56.4 and 56.
#include <type_traits>

#include "jk_ancestors.h"
#include "jk_wave.h"

namespace jk {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

struct FParams {
  const float *q, *kc, *vc, *kt, *vt;
  const int32_t *parent, *prefix_len;
  float* part_o;
  float2* part_ml;
  float* out;     // undivided key range: the result
  unsigned* err;  // the workspace's sticky device error word
  int B, T, Hkv, G, M, m_pad, D, max_prefix, splits;
  long long q_sb, q_st, q_sh, kc_sb, kc_sl, kc_sh, kt_sb, kt_st, kt_sh, o_sb, o_st, o_sh;
  float scale;
};

// KJ: 16-column chunks of a head (rounded up); WAVES: by how many registers that leaves
template <int KJ>
constexpr int waves_for() { return KJ <= 8 ? 8 : 4; }

template <int KJ>
__global__ __launch_bounds__(64 * waves_for<KJ>(), KJ <= 8 ? 2 : 1) void tva_f32_kernel(FParams p) {
  constexpr int WAVES = waves_for<KJ>(), DB = (KJ + 3) / 4, LDO = 64 * DB + 4;
  __shared__ float tops[WAVES][16];     // a wave's maximum of a row,
  __shared__ float2 shares[WAVES][16];  // and its share of the row's sum, beside the maximum of all
  extern __shared__ __attribute__((aligned(16))) float osum[];  // [WAVES][16][LDO]

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int c = lane & 15, g = lane >> 4;
  const int split = blockIdx.x, row0 = blockIdx.y * 16;
  const int kv = blockIdx.z % p.Hkv, b = blockIdx.z / p.Hkv;
  const int D = p.D;
  const float* kc = p.kc + b * p.kc_sb + (long long)kv * p.kc_sh;
  const float* vc = p.vc + b * p.kc_sb + (long long)kv * p.kc_sh;
  const float* kt = p.kt + b * p.kt_sb + (long long)kv * p.kt_sh;
  const float* vt = p.vt + b * p.kt_sb + (long long)kv * p.kt_sh;

  int L = p.prefix_len[b];
  const int pa0 = lane < p.T ? p.parent[(long long)b * p.T + lane] : -1, pa1 = lane + 64 < p.T ? p.parent[(long long)b * p.T + lane + 64] : -1;
  const int m = min(row0 + c, p.M - 1), node = m / p.G;  // this lane's query row (rows past the end repeat the last one)
  floatx4 q[KJ], k[KJ], v[DB][4];  // the row, and a block's K and V
  // column 16 j + 4 g of a row; columns past the end: the row's first ones, against zeros of q
  auto col = [&](int j) { return 16 * j + 4 * g < D ? 16 * j + 4 * g : 0; };
  auto load_k = [&](const float* row) {
#pragma unroll
    for (int j = 0; j < KJ; ++j) k[j] = *reinterpret_cast<const floatx4*>(row + col(j));
  };
  auto load_v = [&](auto v_at) {  // v_at(i): where key i of the block has its values
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float* row = v_at(4 * g + i);
#pragma unroll
      for (int d = 0; d < DB; ++d) v[d][i] = *reinterpret_cast<const floatx4*>(row + (64 * d + 4 * c < D ? 64 * d + 4 * c : 0));
    }
  };
  if (split == 0 && p.max_prefix > 0) load_k(kc + (long long)min(16 * wave + c, p.max_prefix - 1) * p.kc_sl);
  {
    const float* src = p.q + b * p.q_sb + node * p.q_st + (long long)(kv * p.G + m - node * p.G) * p.q_sh;
#pragma unroll
    for (int j = 0; j < KJ; ++j) q[j] = *reinterpret_cast<const floatx4*>(src + col(j));
    if (16 * KJ != D) {
#pragma unroll
      for (int j = 0; j < KJ; ++j)
        if (16 * j + 4 * g >= D) q[j] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
  }
  L = L < 0 ? 0 : (L > p.max_prefix ? p.max_prefix : L);
  const int ktot = L + p.T;  // (at most 512 ranges of at most 65 664 keys)
  const int k_begin = p.splits == 1 ? 0 : (int)((unsigned)split * (unsigned)ktot / (unsigned)p.splits);
  const int k_end = p.splits == 1 ? ktot : (int)((unsigned)(split + 1) * (unsigned)ktot / (unsigned)p.splits);
  const int p_end = min(k_end, L), t_begin = max(k_begin, L);
  const int n_prefix = p_end > k_begin ? (p_end - k_begin + 15) / 16 : 0, n_tree = k_end > t_begin ? (k_end - t_begin + 15) / 16 : 0;

  // The waves with fewer blocks of the prefix take the tree's first; who has one makes its rows' ancestors while the keys come
  const int first = (wave + WAVES - n_prefix % WAVES) % WAVES;
  dev::Ancestors seen{0ull, 0ull};
  if (first < n_tree || (split == 0 && wave == 0)) seen = dev::ancestors_of(p.T, p.err, pa0, pa1, node, split == 0 && row0 == 0 && kv == 0 && wave == 0);

  // A weight of zero - an unseen key's above all - leaves its value out, whatever that is.  The matrix product has one
  // value for sixteen rows' weights, so an infinity or a NaN reaches them all; it stays in the accumulators to the end, and
  // a wave that finds one there takes its keys once more, key by key.  (Looked for in the values themselves, in front of
  // each product: 57.0 us for 4 sequences, 8 heads of 128, 52 nodes, 2100 keys became 59.8.)
  floatx4 o[DB][4];
  float mx, sum;
  // 16 keys, whose K and V have been asked for: visible(i) whether this lane's row sees key 4 g + i; `next` asks for the K of
  // the block behind this one as soon as this one's is used.  (careful: V at v_at(i))
  auto block = [&](auto careful, auto v_at, auto visible, auto next) {
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
    next();
#pragma unroll
    for (int i = 0; i < 4; ++i) s[i] = visible(i) ? s[i] * p.scale : -INFINITY;
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
        const float* row = v_at(key);
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
      return;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int d = 0; d < DB; ++d)
#pragma unroll
        for (int e = 0; e < 4; ++e) o[d][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[d][i][e], s[i], o[d][e], 0, 0, 0);
  };
  auto prefix_k = [&](int blk) { load_k(kc + (long long)min(k_begin + 16 * blk + c, p_end - 1) * p.kc_sl); };
  auto pass = [&](auto careful) {
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
      for (int i = 0; i < 4; ++i) o[d][i] = floatx4{0.f, 0.f, 0.f, 0.f};
    mx = -INFINITY;
    sum = 0.f;
    if ((split != 0 || careful) && wave < n_prefix) prefix_k(wave);
    const int tree_begin = t_begin - L, last = k_end - L - 1;
    auto tree_k = [&](int blk) { load_k(kt + (long long)min(tree_begin + 16 * blk + c, last) * p.kt_st); };
    if (wave >= n_prefix && first < n_tree) tree_k(first);
    for (int blk = wave; blk < n_prefix; blk += WAVES) {
      const int key0 = k_begin + 16 * blk, left = p_end - key0 - 4 * g;
      auto v_at = [&](int i) { return vc + (long long)min(key0 + i, p_end - 1) * p.kc_sl; };
      if (!careful) load_v(v_at);
      block(careful, v_at, [&](int i) { return i < left; },
            [&]() {
              if (blk + WAVES < n_prefix) prefix_k(blk + WAVES);
              else if (first < n_tree) tree_k(first);
            });
    }
    const unsigned long long lo = seen.lo, hi = seen.hi;
    for (int blk = first; blk < n_tree; blk += WAVES) {
      const int key0 = tree_begin + 16 * blk, left = last + 1 - key0 - 4 * g;
      auto v_at = [&](int i) { return vt + (long long)min(key0 + i, last) * p.kt_st; };
      if (!careful) load_v(v_at);
      // the bits of keys key0 .. key0 + 63, then this lane's four
      const unsigned long long set = key0 >= 64 ? hi >> (key0 - 64) : key0 > 0 ? lo >> key0 | hi << (64 - key0) : lo;
      const unsigned mine = (unsigned)(set >> (4 * g));
      block(careful, v_at, [&](int i) { return i < left && ((mine >> i) & 1u); },
            [&]() {
              if (blk + WAVES < n_tree) tree_k(blk + WAVES);
            });
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
      const int n = row / p.G;
      float* dst = p.out + b * p.o_sb + n * p.o_st + (long long)(kv * p.G + row - n * p.G) * p.o_sh;
      const float inv = 1.f / tot;  // (tot > 0: every row sees at least its own tree key)
      *reinterpret_cast<floatx4*>(dst + 4 * x) = floatx4{t[0] * inv, t[1] * inv, t[2] * inv, t[3] * inv};
    } else {
      const long long prow = ((long long)(b * p.Hkv + kv) * p.splits + split) * p.m_pad + row;
      *reinterpret_cast<floatx4*>(p.part_o + prow * D + 4 * x) = t;
      if (x == 0) p.part_ml[prow] = make_float2(shares[0][r].y, tot);
    }
  }
}

template <int KJ>
hipError_t launch_kj(const FParams& fp, hipStream_t stream) {
  constexpr int WAVES = waves_for<KJ>(), SMEM = WAVES * 16 * (64 * ((KJ + 3) / 4) + 4) * 4;
  static LdsLimitRaised raised;
  if (hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(tva_f32_kernel<KJ>), SMEM, raised); e != hipSuccess) return e;
  hipLaunchKernelGGL(tva_f32_kernel<KJ>, dim3(fp.splits, (fp.M + 15) / 16, fp.B * fp.Hkv), dim3(64 * WAVES), SMEM, stream, fp);
  return hipGetLastError();
}

}  // namespace

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
  const jk_attn_desc& d = a.d;
  fp.B = d.batch; fp.T = d.n_tree; fp.Hkv = d.n_kv_heads; fp.G = d.n_q_heads / d.n_kv_heads;
  fp.M = pl.m_rows; fp.m_pad = pl.m_pad; fp.D = d.head_dim; fp.max_prefix = a.max_prefix_len;
  fp.splits = pl.parts;
  fp.q_sb = d.q_stride_b; fp.q_st = d.q_stride_t; fp.q_sh = d.q_stride_h;
  fp.kc_sb = d.kc_stride_b; fp.kc_sl = d.kc_stride_l; fp.kc_sh = d.kc_stride_h;
  fp.kt_sb = d.kt_stride_b; fp.kt_st = d.kt_stride_t; fp.kt_sh = d.kt_stride_h;
  fp.out = static_cast<float*>(a.out);
  fp.o_sb = d.o_stride_b; fp.o_st = d.o_stride_t; fp.o_sh = d.o_stride_h;
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
