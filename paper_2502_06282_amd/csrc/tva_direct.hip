// Tree-masked verification attention, bf16, for calls of few keys (gfx950): K and V straight into registers.
//
// Same definition as tva_bf16.hip.  What bounds a call of a few hundred keys is no rate but a launch, the trips to memory one
// behind the other and the instructions of lone waves between them.  So there is one trip: a wave asks for its page ids, the
// length, its query rows and the K and V of its first block together, on the assumption that the length is the host's bound;
// and there is little to execute: 16 rows a workgroup, no LDS ring, no barrier before the waves' results meet, an undivided key
// range and no second launch.  S^T = K Q^T on v_mfma_f32_16x16x32_bf16 leaves a lane with eight keys of one row, which is what
// O^T = V^T P^T takes as its operand, so the weights stay in their registers.  A lane fetches 16 bytes of each of those eight
// keys of V (whole rows across 16 lanes), and v_perm_b32 puts two keys of a column side by side: 32 of them a block, in place
// of a transposed copy in LDS.
//
// Every row tile draws K and V through its CU (some 67 bytes per ns), so with many keys or rows the kernels that share them
// through LDS are faster: the line between them is the plan's estimate (PlanModel in api.cpp).  Measured, us, the other kernels
// / this one: one sequence, 14 nodes, 32 heads, 36 keys 7.4 / 4.8; 19 sequences, 9 nodes, 16 heads on 2, 36 keys 7.6 / 5.2;
// 8 sequences, 11 nodes, 32 heads on 8, 202 keys 9.0 / 6.0; 2 sequences, 32 nodes, 64 heads on 8, 289 keys 10.0 / 6.9; 400 drawn
// calls of up to 900 keys 0.856 in the geometric mean.  Error against fp64 1.9 - 2.3e-3 of the norm (the others 1.9 - 2.9e-3).
// With 32 rows a workgroup every call took 1.5 - 2 us more (twice the instructions at its start and end); with eight waves
// calls of few keys took the same and those of many workgroups up to half as long again; splits of the keys over workgroups,
// merged by the last to come, paid for themselves in 3 of 60 calls.
#include "jk_ancestors.h"
#include "jk_wave.h"
#include "tva_tiles.h"

namespace jk {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

template <int D>
struct VRow {  // 16 lanes' shares of a row of V
  typedef u32x4 type;
};
template <>
struct VRow<64> {
  typedef u32x2 type;
};

// 16 query rows of one (sequence, KV head) a workgroup; its waves take blocks of 32 keys in turn
constexpr int kRows = 16, kWaves = 4;

template <int D, bool PAGED>
__global__ __launch_bounds__(64 * kWaves, 2) void tva_direct_kernel(const KParams p) {
  constexpr int DJ = D / 32, E = D / 16, LDO = D + 4;
  typedef typename VRow<D>::type v_row;
  __shared__ float tops[kWaves][kRows];                                            // a wave's maximum of a row (log2 units),
  __shared__ float shares[kWaves][kRows];                                          // its share of the row's sum,
  __shared__ __attribute__((aligned(16))) float osum[kWaves][kRows][LDO];  // and of the row

  {  // every 64-byte line of the kernel arguments at once: the compiler fetches them in several dependent batches
    typedef __attribute__((address_space(4))) const unsigned kernarg_word;
    kernarg_word* ka = (kernarg_word*)__builtin_amdgcn_kernarg_segment_ptr();
    static_assert(sizeof(KParams) > 320 && sizeof(KParams) <= 384, "six lines of kernel arguments");
    const unsigned a0 = ka[0], a1 = ka[16], a2 = ka[32], a3 = ka[48], a4 = ka[64], a5 = ka[80];
    asm volatile("" ::"s"(a0), "s"(a1), "s"(a2), "s"(a3), "s"(a4), "s"(a5));
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, g = lane >> 4;
  const int T = p.T, G = p.G, M = p.M;
  // Consecutive workgroups alternate between the XCDs: each XCD has a range of the row tiles, the tiles of one (sequence, KV
  // head) side by side, so that they share its K and V.
  const int tile = (blockIdx.x & 7) * (p.total_wgs >> 3) + (blockIdx.x >> 3);
  const int unit = div_mg(tile, p.mg_qtiles), row0 = (tile - unit * p.n_qtiles) * kRows;
  if (unit >= p.B * p.Hkv) return;  // padding
  const int b = div_mg(unit, p.mg_hkv), kv = unit - b * p.Hkv;

  int lane_zero = 0;
  asm volatile("" : "+v"(lane_zero));  // (a vector load: a scalar one would be waited for with the arguments)
  const int L_raw = __hip_atomic_load(p.prefix_len + b + lane_zero, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

  // ---- this wave's blocks of 32 keys: wave + 4 i, the prefix's in front of the tree's
  const int n_tblk = (T + kTileKeys - 1) / kTileKeys;
  int L = p.max_prefix, n_pblk = (L + kTileKeys - 1) / kTileKeys;
  // page ids of 64 blocks of this wave, a lane each; ids outside the pool are clamped (and reported where they count)
  int ids = 0;
  auto ask_pages = [&](int first) {
    const int blk = first + kWaves * lane, at = div_mg(blk, p.mg_tpp);
    ids = blk < n_pblk && at < p.max_blocks ? p.block_table[(long long)b * p.max_blocks + at] : 0;
  };
  if (PAGED) ask_pages(wave);

  const int m = min(row0 + c, M - 1), node = div_mg(m, p.mg_g);  // this lane's query row (rows past the end repeat the last one)
  bf16x8 q[DJ];
  if (wave < n_pblk + n_tblk) {  // (the rows of a wave without keys would only stand in the others' way)
    const uint16_t* src = p.q + b * p.q_sb + node * p.q_st + (long long)(kv * G + (m - node * G)) * p.q_sh + 8 * g;
#pragma unroll
    for (int j = 0; j < DJ; ++j) q[j] = *reinterpret_cast<const bf16x8*>(src + 32 * j);
  }
  const int pa0 = lane < T ? p.parent[(long long)b * T + lane] : -1;
  const int pa1 = lane + 64 < T ? p.parent[(long long)b * T + lane + 64] : -1;

  bf16x8 k[2][DJ];
  v_row v[8];
  const uint16_t* kc = p.kc + (PAGED ? 0 : b * p.kc_sb) + (long long)kv * p.kc_sh;
  const uint16_t* vc = p.vc + (PAGED ? 0 : b * p.kc_sb) + (long long)kv * p.kc_sh;
  const uint16_t* kt = p.kt + b * p.kt_sb + (long long)kv * p.kt_sh;
  const uint16_t* vt = p.vt + b * p.kt_sb + (long long)kv * p.kt_sh;
  // A lane has keys c and 16 + c of K (8 columns of each 32), and of V columns (D / 16) c .. of keys 4 g + i and 16 + 4 g + i:
  // the ones whose scores S^T = K Q^T leaves with it.
  struct Block {
    long long at;  // first row, in elements from the cache's (tree's) first
    int stride8;   // row stride / 8
    int last;      // last row that exists
    bool tree;
  };
  auto block_at = [&](int blk) {
    Block x;
    x.tree = blk >= n_pblk;
    if (x.tree) {
      x.at = (long long)(blk - n_pblk) * kTileKeys * p.kt_st;
      x.stride8 = (int)(p.kt_st >> 3);
      x.last = min(kTileKeys, T - (blk - n_pblk) * kTileKeys) - 1;
    } else {
      x.stride8 = (int)(p.kc_sl >> 3);
      x.last = min(kTileKeys, L - blk * kTileKeys) - 1;
      if (PAGED) {
        const int id = __builtin_amdgcn_readlane(ids, (blk / kWaves) & 63), page = id < 0 ? 0 : (id >= p.n_pages ? p.n_pages - 1 : id);
        const int slot = blk - div_mg(blk, p.mg_tpp) * p.tpp;
        x.at = (long long)page * p.page_stride + (long long)slot * kTileKeys * p.kc_sl;
      } else {
        x.at = (long long)blk * kTileKeys * p.kc_sl;
      }
    }
    return x;
  };
  auto off16 = [&](const Block& x, int row) { return __umul24((unsigned)min(row, x.last), (unsigned)x.stride8) << 4; };
  auto load_k = [&](const Block& x) {
    const unsigned char* base = reinterpret_cast<const unsigned char*>(uniform_ptr((x.tree ? kt : kc) + x.at));
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const unsigned off = off16(x, 16 * h + c) + 16u * g;
#pragma unroll
      for (int j = 0; j < DJ; ++j) k[h][j] = *reinterpret_cast<const bf16x8*>(base + off + 64 * j);
    }
  };
  auto load_v = [&](const Block& x) {
    const unsigned char* base = reinterpret_cast<const unsigned char*>(uniform_ptr((x.tree ? vt : vc) + x.at));
#pragma unroll
    for (int i = 0; i < 8; ++i)
      v[i] = *reinterpret_cast<const v_row*>(base + off16(x, (i & 4) * 4 + 4 * g + (i & 3)) + (unsigned)(sizeof(v_row) * c));
  };

  // ---- the first block on the assumption that the length is the host's bound
  Block cur;
  if (wave < n_pblk + n_tblk) {
    cur = block_at(wave);
    load_k(cur);
    load_v(cur);
  }
  {
    const int len = __builtin_amdgcn_readfirstlane(L_raw);
    L = len < 0 ? 0 : (len > p.max_prefix ? p.max_prefix : len);
  }
  if (L != p.max_prefix) {  // (uniform)
    n_pblk = (L + kTileKeys - 1) / kTileKeys;
    if (wave < n_pblk + n_tblk && (wave + 1) * kTileKeys > L) {  // (never more blocks than assumed: its query rows are there)
      cur = block_at(wave);
      load_k(cur);
      load_v(cur);
    }
  }
  const int end = n_pblk + n_tblk;

  dev::Ancestors seen{0ull, 0ull};
  const bool reports = row0 == 0 && kv == 0 && wave == 0;
  if (reports || (wave < end && wave + (end - 1 - wave) / kWaves * kWaves >= n_pblk))  // the wave has a block of the tree
    seen = dev::ancestors_of(T, p.err, pa0, pa1, node, reports);

  floatx4 o[E];
#pragma unroll
  for (int e = 0; e < E; ++e) o[e] = floatx4{0.f, 0.f, 0.f, 0.f};
  float mx = -INFINITY, sum = 0.f;
  bool bad_page = false;
  for (int blk = wave; blk < end; blk += kWaves) {
    if (PAGED && !cur.tree) {
      const int id = __builtin_amdgcn_readlane(ids, (blk / kWaves) & 63);
      bad_page = bad_page || id < 0 || id >= p.n_pages;
    }
    floatx4 s[2] = {floatx4{0.f, 0.f, 0.f, 0.f}, floatx4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int j = 0; j < DJ; ++j)
#pragma unroll
      for (int h = 0; h < 2; ++h) s[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k[h][j], q[j], s[h], 0, 0, 0);
    const Block now = cur;
    const bool more = blk + kWaves < end;
    if (more) {
      if (PAGED && ((blk / kWaves + 1) & 63) == 0) ask_pages(blk + kWaves);
      cur = block_at(blk + kWaves);
      load_k(cur);
    }
    if (now.tree || now.last < kTileKeys - 1) {  // (uniform) which of its keys the row sees: bits 4 g + r and 16 + 4 g + r
      unsigned bits = (2u << now.last) - 1u;
      if (now.tree) {
        const int t = blk - n_pblk;
        bits = (unsigned)((t & 2 ? seen.hi : seen.lo) >> (32 * (t & 1)));
      }
      bits >>= 4 * g;
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int r = 0; r < 4; ++r) s[h][r] = (bits >> (16 * h + r)) & 1u ? s[h][r] : -INFINITY;
    }
    float top = fmaxf(fmaxf(fmaxf(s[0][0], s[0][1]), fmaxf(s[0][2], s[0][3])), fmaxf(fmaxf(s[1][0], s[1][1]), fmaxf(s[1][2], s[1][3])));
    top = fmaxf(top, __uint_as_float(dev::other16(__float_as_uint(top), lane & 16)));
    top = fmaxf(top, __uint_as_float(dev::other32(__float_as_uint(top), lane & 32)));
    top *= p.scale_log2;
    // (the reference moves only when it is exceeded by more than 2^8: weights, their sum and the accumulators all carry it)
    const bool up = top > mx + 8.f;
    const float ref = up ? top : mx, use = ref == -INFINITY ? 0.f : ref;
    if (__any(up && mx != -INFINITY)) {
      const float f = up ? fast_exp2(mx - use) : 1.f;
      sum *= f;
#pragma unroll
      for (int e = 0; e < E; ++e)
#pragma unroll
        for (int r = 0; r < 4; ++r) o[e][r] *= f;
    }
    mx = ref;
    bf16x8 w;  // (the sum takes the rounded weights: numerator and denominator carry the same rounding)
    bf16x2 one;
    one[0] = one[1] = (__bf16)1.f;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int r = 0; r < 4; r += 2) {
        bf16x2 pk;
        pk[0] = (__bf16)fast_exp2(fmaf(s[h][r], p.scale_log2, -use));
        pk[1] = (__bf16)fast_exp2(fmaf(s[h][r + 1], p.scale_log2, -use));
        sum = __builtin_amdgcn_fdot2_f32_bf16(pk, one, sum, false);
        w[4 * h + r] = pk[0];
        w[4 * h + r + 1] = pk[1];
      }
    // O^T += V^T P^T, a column of each lane's at a time: its eight keys side by side
#pragma unroll
    for (int e = 0; e < E; ++e) {
      u32x4 a;
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = __builtin_amdgcn_perm(v[2 * i + 1][e / 2], v[2 * i][e / 2], e & 1 ? 0x07060302u : 0x05040100u);
      o[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), w, o[e], 0, 0, 0);
    }
    if (more) load_v(cur);
  }
  if (PAGED && bad_page && lane == 0) __hip_atomic_fetch_or(p.err, kDevErrBadPage, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

  // ---- the waves' shares of a row meet, each scaled by its own wave
  const int used = min(kWaves, end);  // waves that have had keys
  sum += __uint_as_float(dev::other16(__float_as_uint(sum), lane & 16));
  sum += __uint_as_float(dev::other32(__float_as_uint(sum), lane & 32));
  if (g == 0) tops[wave][c] = mx;
  constexpr int LPR = D / 8;  // a thread has eight columns of one row of the result
  static_assert(kRows * LPR <= 64 * kWaves, "all of them at once");
  const int r = tid / LPR, x8 = tid % LPR * 8, row = row0 + r, nd = div_mg(min(row, M - 1), p.mg_g);
  uint16_t* dst = p.out + b * p.o_sb + nd * p.o_st + (long long)(kv * G + (row - nd * G)) * p.o_sh + x8;
  __syncthreads();
  if (wave < used) {
    float all = tops[0][c];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) all = fmaxf(all, tops[w][c]);  // (-inf of a wave without keys)
    const float f = mx == -INFINITY ? 0.f : fast_exp2(mx - all);
    if (g == 0) shares[wave][c] = sum * f;
    float* to = &osum[wave][c][(D / 4) * g];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int e = 0; e < E; e += 4)
        *reinterpret_cast<floatx4*>(to + E * i + e) = floatx4{o[e][i] * f, o[e + 1][i] * f, o[e + 2][i] * f, o[e + 3][i] * f};
  }
  __syncthreads();
  if (r >= kRows || row >= M) return;
  floatx4 t0 = {0.f, 0.f, 0.f, 0.f}, t1 = t0;
  float tot = 0.f;
#pragma unroll
  for (int w = 0; w < kWaves; ++w)
    if (w < used) {
      t0 += *reinterpret_cast<const floatx4*>(&osum[w][r][x8]);
      t1 += *reinterpret_cast<const floatx4*>(&osum[w][r][x8 + 4]);
      tot += shares[w][r];
    }
  const float inv = 1.f / tot;  // (every row sees at least its own tree key)
  u32x4 out;
  out[0] = dev::pack_bf16(t0[0] * inv, t0[1] * inv);
  out[1] = dev::pack_bf16(t0[2] * inv, t0[3] * inv);
  out[2] = dev::pack_bf16(t1[0] * inv, t1[1] * inv);
  out[3] = dev::pack_bf16(t1[2] * inv, t1[3] * inv);
  dev::store_through(dst, out);
}

}  // namespace

namespace tva {
hipError_t launch_direct(const KParams& kp, int head_dim, hipStream_t stream) {
  const dim3 grid(kp.total_wgs), block(64 * kWaves);
  const bool paged = kp.block_table != nullptr;
  if (head_dim == 128 && paged) hipLaunchKernelGGL((tva_direct_kernel<128, true>), grid, block, 0, stream, kp);
  else if (head_dim == 128) hipLaunchKernelGGL((tva_direct_kernel<128, false>), grid, block, 0, stream, kp);
  else if (head_dim == 64 && paged) hipLaunchKernelGGL((tva_direct_kernel<64, true>), grid, block, 0, stream, kp);
  else if (head_dim == 64) hipLaunchKernelGGL((tva_direct_kernel<64, false>), grid, block, 0, stream, kp);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}
}  // namespace tva

}  // namespace jk
