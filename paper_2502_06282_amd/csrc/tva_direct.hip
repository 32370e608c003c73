// Tree-masked verification attention, bf16, for calls of few keys (gfx950): K and V straight into registers.
//
// Same definition as tva_bf16.hip.  What bounds a call of a few hundred keys is no rate but a launch, the trips to memory one
// behind the other and the instructions of lone waves between them (8 cycles each where one waits for the other).  So there is
// one trip: a wave asks for its page ids, the length, its query rows and the K and V of its first block together, on the
// assumption that the length is the host's bound; a tree's blocks come first, so that a shorter length changes nothing of that.
// None of it is asked for in a branch, and all of it by loads that count as nothing else: behind a branch, and with flat loads,
// the compiler waited for K and V where it waited for the length (0.5 - 0.8 us of every call).  And there is little to execute:
// 16 rows a workgroup, no LDS ring, no barrier before the waves' results meet, an undivided key range and no second launch.
// S^T = K Q^T on v_mfma_f32_16x16x32_bf16 leaves a lane with eight keys of one row, which is what O^T = V^T P^T takes as its
// operand, so the weights stay in their registers.  A lane fetches 16 bytes of each of those eight keys of V (whole rows across 16
// lanes), and v_perm_b32 puts two keys of a column side by side: 32 of them a block, in place of a transposed copy in LDS.
//
// Every row tile draws K and V through its CU (some 60 bytes per ns), so with many keys or rows the kernels that share them
// through LDS are faster: the line between them is the plan's estimate (PlanModel in api.cpp).  Measured, us, the other kernels
// / this one with flat loads and branches / like this: one sequence, 14 nodes, 32 heads, 36 keys 6.3 / 4.8 / 4.1; 19 sequences, 9
// nodes, 16 heads on 2, 36 keys 6.8 / 5.2 / 4.1; 8 sequences, 11 nodes, 32 heads on 8, 202 keys 9.0 / 6.0 / 5.7; 2 sequences, 32
// nodes, 64 heads on 8, 289 keys 10.1 / 6.9 / 6.7; 320 drawn calls of 80 - 1300 keys 1 / 0.85 / 0.84 in the geometric mean.
// Error against fp64 2.0 - 2.2e-3 of the norm (the others 1.9 - 2.9e-3).  With 32 rows a workgroup every call took 1.5 - 2 us more
// (twice the instructions at its start and end); with eight waves calls of few workgroups took 0 - 0.9 us more and those of many up
// to half as long again; splits of the keys over workgroups, merged by the last to come, paid for themselves in 3 of 60 calls.
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

// Addresses that are known to be in device memory: made from a pointer in scalar registers, a load is otherwise a flat one, which
// counts as an access to LDS as well and takes its 64-bit address from two vector registers
typedef __attribute__((address_space(1))) const unsigned char device_bytes;
__device__ __forceinline__ device_bytes* in_device(const uint16_t* p) { return (device_bytes*)(unsigned long long)uniform_ptr(p); }
template <class T>
__device__ __forceinline__ T load_at(device_bytes* base, unsigned off) {
  return *(__attribute__((address_space(1))) const T*)(base + off);
}

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

  // ---- this wave's blocks of 32 keys: wave + kWaves * i, the tree's in front of the prefix's, so that what a wave asks for
  // first does not depend on the length
  const int n_tblk = (T + kTileKeys - 1) / kTileKeys;
  int L = p.max_prefix, n_pblk = (L + kTileKeys - 1) / kTileKeys;
  const bool some = wave < n_tblk + n_pblk;  // (the length's bound)
  // What is asked for here is asked for without a branch: the compiler waits for everything behind a load that it may have passed
  // by.  A wave without keys asks for one address in all lanes.
  const int tc = some ? c : 0, tg = some ? g : 0;
  const int pa_lo = p.parent[(long long)b * T + min(lane, T - 1)], pa_hi = p.parent[(long long)b * T + min(lane + 64, T - 1)];
  // page ids of 64 blocks of this wave, a lane each; ids outside the pool are clamped (and reported where they count).  (A planned
  // call has at most 28 blocks for all waves; only where this kernel is forced are there more than one lane each.)
  int ids = 0;
  auto ask_pages = [&](int first) {
    const int at = div_mg(max(first + kWaves * lane - n_tblk, 0), p.mg_tpp);
    ids = p.block_table[(long long)b * p.max_blocks + min(at, p.max_blocks - 1)];
  };
  if (PAGED) ask_pages(wave);

  const int m = min(row0 + c, M - 1), node = div_mg(m, p.mg_g);  // this lane's query row (rows past the end repeat the last one)
  bf16x8 q[DJ];
  {
    const int tm = some ? m : row0, tn = some ? node : div_mg(row0, p.mg_g);
    const uint16_t* src = p.q + b * p.q_sb + tn * p.q_st + (long long)(kv * G + (tm - tn * G)) * p.q_sh + 8 * tg;
#pragma unroll
    for (int j = 0; j < DJ; ++j) q[j] = *reinterpret_cast<const bf16x8*>(src + 32 * j);
  }

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
    x.tree = blk < n_tblk;
    if (x.tree) {
      x.at = (long long)blk * kTileKeys * p.kt_st;
      x.stride8 = (int)(p.kt_st >> 3);
      x.last = min(kTileKeys, T - blk * kTileKeys) - 1;
    } else {
      const int pb = blk - n_tblk;
      x.stride8 = (int)(p.kc_sl >> 3);
      x.last = min(kTileKeys, L - pb * kTileKeys) - 1;
      if (PAGED) {
        const int id = __builtin_amdgcn_readlane(ids, (blk / kWaves) & 63), page = id < 0 ? 0 : (id >= p.n_pages ? p.n_pages - 1 : id);
        const int slot = pb - div_mg(pb, p.mg_tpp) * p.tpp;
        x.at = (long long)page * p.page_stride + (long long)slot * kTileKeys * p.kc_sl;
      } else {
        x.at = (long long)pb * kTileKeys * p.kc_sl;
      }
    }
    return x;
  };
  auto off16 = [&](const Block& x, int row) { return __umul24((unsigned)min(row, x.last), (unsigned)x.stride8) << 4; };
  auto load_k = [&](const Block& x, int c, int g) {
    device_bytes* base = in_device((x.tree ? kt : kc) + x.at);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const unsigned off = off16(x, 16 * h + c) + 16u * g;
#pragma unroll
      for (int j = 0; j < DJ; ++j) k[h][j] = load_at<bf16x8>(base, off + 64 * j);
    }
  };
  auto load_v = [&](const Block& x, int c, int g) {
    device_bytes* base = in_device((x.tree ? vt : vc) + x.at);
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = load_at<v_row>(base, off16(x, (i & 4) * 4 + 4 * g + (i & 3)) + (unsigned)(sizeof(v_row) * c));
  };

  // ---- the first block on the assumption that the length is the host's bound
  Block cur = block_at(some ? wave : 0);
  if (!some) cur.stride8 = 0;
  load_k(cur, tc, tg);
  load_v(cur, tc, tg);
  {
    const int len = __builtin_amdgcn_readfirstlane(L_raw);
    L = len < 0 ? 0 : (len > p.max_prefix ? p.max_prefix : len);
  }
  n_pblk = (L + kTileKeys - 1) / kTileKeys;
  if (!cur.tree) cur.last = min(kTileKeys, L - (wave - n_tblk) * kTileKeys) - 1;  // (below zero: no block any more)
  const int end = n_pblk + n_tblk;

  dev::Ancestors seen{0ull, 0ull};
  const bool reports = row0 == 0 && kv == 0 && wave == 0;
  if (reports || wave < n_tblk)  // the wave has a block of the tree
    seen = dev::ancestors_of(T, p.err, lane < T ? pa_lo : -1, lane + 64 < T ? pa_hi : -1, node, reports);

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
      load_k(cur, c, g);
    }
    if (now.tree || now.last < kTileKeys - 1) {  // (uniform) which of its keys the row sees: bits 4 g + r and 16 + 4 g + r
      unsigned bits = (2u << now.last) - 1u;
      if (now.tree) {
        bits = (unsigned)((blk & 2 ? seen.hi : seen.lo) >> (32 * (blk & 1)));
      }
      bits >>= 4 * g;
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int r = 0; r < 4; ++r) s[h][r] = (bits >> (16 * h + r)) & 1u ? s[h][r] : -INFINITY;
      if (!now.tree) {  // (asked for beyond the prefix's end: what is there may be no number)
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = (i & 4) * 4 + 4 * g + (i & 3) <= now.last ? v[i] : v_row{};
      }
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
    if (more) load_v(cur, c, g);
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
  if (head_dim == 128)
    return paged ? launch_kernel(tva_direct_kernel<128, true>, grid, block, 0, stream, kp)
                 : launch_kernel(tva_direct_kernel<128, false>, grid, block, 0, stream, kp);
  if (head_dim == 64)
    return paged ? launch_kernel(tva_direct_kernel<64, true>, grid, block, 0, stream, kp)
                 : launch_kernel(tva_direct_kernel<64, false>, grid, block, 0, stream, kp);
  return hipErrorInvalidValue;
}
}  // namespace tva

}  // namespace jk
