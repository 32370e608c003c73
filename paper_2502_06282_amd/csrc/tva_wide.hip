// Tree-masked verification attention, bf16 inputs, 64 query rows per wave (gfx950): the kernel of calls with many query
// rows per KV head and long key ranges.  The problem, the packing of query rows, the tiles and their swizzles are those of
// tva_bf16.hip; this one differs in how much a wave holds and in how it fills its SIMD.
//
// A workgroup of four waves has 256 query rows and a CU to itself: a wave holds two blocks of 32 rows, their queries and
// accumulators (192 of its 512 registers), and every K or V operand read from LDS serves both.  With 32 rows per wave the
// operand reads alone ask for all of the LDS bandwidth that a matrix pipe at full rate leaves (1 KB per 32 cycles and
// SIMD), and every 128 rows stream K and V once more.
//
// A tile of 32 keys takes two phases.  In each the score product of one block, the value product of one block and the
// softmax of one block run side by side, all independent of each other:
//     A(t):  S1(t)    O1 += V(t-1) P1(t-1)    softmax of S0(t)
//     B(t):  S0(t+1)  O0 += V(t)   P0(t)      softmax of S1(t)
// written out slot by slot: a matrix instruction of 32 cycles, and the vector instructions and LDS reads that a lone wave
// can issue beside it (about six).  K(t+1) and V(t) are read over the registers of K(t) and V(t-1) once those are used up.
// What a slot may hold was measured (a lone wave per SIMD, cycles per 16 slots of 32): with a fused multiply-add, an
// exponential and an addition 532; a bf16 dot product among them 796 (it runs on the matrix pipe, and not beside it).  So
// a row's sum is one more matrix product: v_mfma_f32_16x16x32_bf16 with a matrix that adds up the eight weights of a lane
// and of its partner in the other half-wave (16 cycles for 512 weights), of the weights as they are rounded.
//
// What bounds it: the vector instructions beside the matrix instructions, and the clock, which the card lowers under this
// load (1.5 to 1.9 GHz: with all of K and V in the caches a tile takes 0.88 us, with them in memory 0.9 - 1.0).  A tile takes 1330 cycles, of which 1120 are matrix instructions.  Measured against the kernel of
// four waves with 32 rows: 8 sequences of 16384 keys, 8 KV heads, 800 rows 476 -> 399 us; 16 sequences of at most 4096 keys
// in pages, 8 KV heads, 240 rows 70 -> 59 us; 29 sequences of 10023 keys, 46 nodes, D = 64 255 -> 178 us.
#include <type_traits>

#include "jk_wave.h"
#include "tva_tiles.h"
#include "tva_wide_order.h"

namespace jk {
namespace {
using tva::KParams;

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kWideThreads = 256, kWideWaves = 4, kBlocks = 2, kWideRows = kBlocks * kWaveRows;

template <int D, bool PAGED>
struct WidePlan {
  using G_ = Geo<D>;
  static constexpr int HALF_BYTES = 64 * 1024;                   // K's half of the ring, in front of V's
  static constexpr int NR = HALF_BYTES / G_::TILE_BYTES;         // tiles in the ring: 8 (D = 128) or 16
  static constexpr int AHEAD = tva::wide_ahead(D);               // tiles asked for in front of the one in use
  static constexpr int RING_BYTES = 2 * HALF_BYTES;
  static constexpr int QROWS = kWideWaves * kWideRows;
  static constexpr int PATCH_LD = D * 2 + 16;                    // padded row of the store patches (after the loop)
  static constexpr int PATCH_BYTES = kWaveRows * PATCH_LD;
  static constexpr int PAGES_BYTES = PAGED ? kMaxPagesPerSplit * 4 : 0;
  static constexpr int DUMP_BYTES = 2 * G_::TILE_BYTES;          // where transfers go that nobody needs
  static constexpr int SMEM = RING_BYTES + DUMP_BYTES + JK_MAX_TREE * 16 + JK_MAX_TREE * 4 + 16 + PAGES_BYTES;
  static_assert(kWideWaves * PATCH_BYTES <= RING_BYTES && SMEM <= 160 * 1024 && AHEAD == NR - 1, "LDS plan");
};

// What a wave holds: two blocks of 32 query rows (a lane has row lane % 32 of each), and the operands in flight
template <int D>
struct WideState {
  static constexpr int DK = Geo<D>::DK, DB = Geo<D>::DB;
  bf16x8 q[kBlocks][DK];
  floatx16 o[kBlocks][DB];
  floatx4 l[kBlocks];       // row sums (four times the same)
  float m[kBlocks], mu[kBlocks];  // reference of the row's weights in log2 units; 0 instead of -inf
  floatx16 s[kBlocks];      // scores
  floatx16 x[kBlocks];      // weights in fp32, on their way
  bf16x8 p[kBlocks][2];     // weights in bf16: operands of the value product
  bf16x8 kf[DK], vf[2 * DB];
  bf16x8 adds;              // the matrix that adds up weights (see row_sums)
};

// One phase.  X: the block whose scores are computed (of K in st.kf); Y: the block whose output takes V (st.vf) times its
// weights; Z: the block whose softmax runs.  A: X = Y = 1, Z = 0; B: X = Y = 0, Z = 1.  The softmax of element e of a
// block: fma in slot e / EPS of its phase, exponential one later, rounding two later, the sums four later; what lies
// past the phase's end runs in the next phase.  `reads(slot)`: LDS reads (over operands that the slots so far have used
// up) and transfers.
template <int D, int Z>
__device__ __forceinline__ void softmax_slot(WideState<D>& st, int slot, float scale_log2) {
  constexpr int NS = 2 * WideState<D>::DK, EPS = 16 / NS;  // slots of a phase; elements a slot
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int at = e / EPS;
    if (slot == at) st.x[Z][e] = fmaf(st.s[Z][e], scale_log2, -st.mu[Z]);
    if (slot == at + 1) st.x[Z][e] = fast_exp2(st.x[Z][e]);
    if ((e & 1) && slot == at + 2) {
      bf16x2 two;
      two[0] = (__bf16)st.x[Z][e - 1];
      two[1] = (__bf16)st.x[Z][e];
      unsigned w = __builtin_bit_cast(unsigned, two);
      asm volatile("" : "+v"(w));  // (rounded here: left alone, the compiler rounds all eight weights of an operand at once)
      u32x4 all = __builtin_bit_cast(u32x4, st.p[Z][e / 8]);
      all[e % 8 / 2] = w;
      st.p[Z][e / 8] = __builtin_bit_cast(bf16x8, all);
    }
    if (e % 8 == 7 && slot == at + 4) st.l[Z] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(st.adds, st.p[Z][e / 8], st.l[Z], 0, 0, 0);
  }
}
template <int D, int Z>
__device__ __forceinline__ void softmax_rest(WideState<D>& st, float scale_log2) {  // past the phase's end
  constexpr int NS = 2 * WideState<D>::DK;
#pragma unroll
  for (int slot = NS; slot < NS + 4; ++slot) softmax_slot<D, Z>(st, slot, scale_log2);
}
template <int D, int X, class Reads>
__device__ __forceinline__ void phase(WideState<D>& st, float scale_log2, const Reads& reads) {
  constexpr int DK = WideState<D>::DK, DB = WideState<D>::DB, NS = 2 * DK, Z = 1 - X;
  static_assert(2 * DB == DK, "as many value products as score products");
#pragma unroll
  for (int slot = 0; slot < NS; ++slot) {
    const int h = slot / 2;
    if (slot % 2 == 0) {
      const floatx16 zero = {};
      st.s[X] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(st.kf[h], st.q[X][h], h == 0 ? zero : st.s[X], 0, 0, 0);
    } else {
      st.o[X][h % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(st.vf[h], st.p[X][h / DB], st.o[X][h % DB], 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    reads(slot);
    if (slot < 4) softmax_slot<D, X>(st, NS + slot, scale_log2);
    softmax_slot<D, Z>(st, slot, scale_log2);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// x / d, both positive, x below 2^20: half a unit keeps the quotient away from whole numbers by more than its error
__device__ __forceinline__ int divided(int x, int d) { return (int)(((float)x + 0.5f) * __builtin_amdgcn_rcpf((float)d)); }

// Paged cache: how far tile `i` of the piece, a full prefix tile, lies behind the pool's start, one tile per lane
struct PagedTile {
  long long at;
  __device__ __forceinline__ long long offset(int lane) const {
    const unsigned lo = __builtin_amdgcn_readlane((int)at, lane), hi = __builtin_amdgcn_readlane((int)(at >> 32), lane);
    return (long long)((unsigned long long)hi << 32 | lo);
  }
};
__device__ __forceinline__ PagedTile paged_tile(const TileSrc& ts, int i, float inv_tpp) {
  const int t = ts.t_begin + i, pi = (int)(((float)t + 0.5f) * inv_tpp);  // (see `divided`)
  PagedTile p;
  p.at = (long long)ts.pg_s[pi - ts.pg_first] * ts.page_stride + (long long)((t - pi * ts.tpp) * kTileKeys) * ts.kc_sl;
  return p;
}

// A batch of `batch` (at most 64) sequences is cut into at most batch * splits pieces (per KV head) of equal length, as
// nearly as whole pieces of whole sequences allow: the pieces are as short as they can be without being more.  Lane b
// brings sequence b's tiles, and gets the number of its first piece and of its pieces.  64 lengths are tried at once: from
// the mean piece to a `splits`th of the longest sequence, which always does (and keeps a paged cache's pieces as short as
// the host assumes).
struct Deal {
  int first, pieces;
};
__device__ __forceinline__ Deal deal_pieces(int tiles, int batch, int splits, int lane) {
  // (Nothing else runs yet, and a call waits for these instructions: four sequences at a time, which those past the batch's
  // end, without tiles, do not change.)
  const int places = batch * splits;
  const float total = dev::wave_sum((float)tiles);
  const int longest = __builtin_amdgcn_readfirstlane((int)dev::wave_max((float)tiles));  // (below 2^20: exact)
  const int hi = divided(longest + splits - 1, splits);
  const int lo = min(max((int)(total * __builtin_amdgcn_rcpf((float)places)), 1), hi);
  const int len = lane == 63 ? hi : lo + (int)((float)(hi - lo) * (float)lane * (1.f / 63.f));
  // (tiles / len rounded up as in `divided`, the half unit and len - 1 brought along by the addition; without tiles 0, as len - 1/2 is less
  // than len.  The quotient's error is below a quarter of a millionth of it, tiles and len together below 2^20: not half a unit.)
  struct Cut {
    float inv, up;
    __device__ __forceinline__ explicit Cut(int len) : inv(__builtin_amdgcn_rcpf((float)len)), up(((float)len - 0.5f) * inv) {}
    __device__ __forceinline__ int pieces(float tiles) const { return (int)fmaf(tiles, inv, up); }
  };
  const Cut cut(len);
  const float tiles_f = (float)tiles;
  int count = 0;
  for (int i = 0; i < batch; i += 4)
#pragma unroll
    for (int k = 0; k < 4; ++k)
      count += cut.pieces(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(tiles_f), i + k)));
  const int best = __builtin_amdgcn_readlane(len, __ffsll((long long)__ballot(count <= places)) - 1);
  Deal d;
  d.pieces = Cut(best).pieces(tiles_f);  // (the same operations: all together as many as were counted)
  // (sums over the lanes in front: by lane moves.  Sequence by sequence the loop had a branch for each of them, and dealing sixteen took
  // 1.75 us at the clock of a loaded card, 0.9 like this.)
  d.first = dev::wave_scan(d.pieces) - d.pieces;
  return d;
}

template <int D, bool PAGED>
__global__ __launch_bounds__(kWideThreads, 1) void tva_wide_kernel(const KParams p) {
  using G_ = Geo<D>;
  using P_ = WidePlan<D, PAGED>;
  constexpr int DK = G_::DK, DB = G_::DB, NR = P_::NR, TILE_BYTES = G_::TILE_BYTES, QROWS = P_::QROWS;
  constexpr int N = LaneChunks<D, kWideWaves>::N;  // transfers of a wave per tile

  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];  // the kernel has no other LDS: offset 0
  unsigned long long* anc = reinterpret_cast<unsigned long long*>(smem + P_::RING_BYTES + P_::DUMP_BYTES);  // [128][2]
  int* par_s = reinterpret_cast<int*>(anc + 2 * JK_MAX_TREE);                                               // [128]
  int* repeat_s = par_s + JK_MAX_TREE;  // set by a wave whose scores left the fixed reference frame
  int* pg_s = repeat_s + 4;             // [1024], paged caches only

  {  // (every line of the kernel arguments asked for at once)
    typedef __attribute__((address_space(4))) const unsigned kernarg_word;
    kernarg_word* ka = (kernarg_word*)__builtin_amdgcn_kernarg_segment_ptr();
    static_assert(sizeof(KParams) > 320 && sizeof(KParams) <= 384, "six lines of kernel arguments");
    const unsigned a0 = ka[0], a1 = ka[16], a2 = ka[32], a3 = ka[48], a4 = ka[64], a5 = ka[80];
    asm volatile("" ::"s"(a0), "s"(a1), "s"(a2), "s"(a3), "s"(a4), "s"(a5));
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c32 = lane & 31, g = lane >> 5;
  const int T = p.T, G = p.G, M = p.M, splits = p.splits;
  const float scale_log2 = p.scale_log2;

  // ---- which piece of work: each XCD a contiguous range of logical ids, the row tiles of one piece side by side.  One
  // sequence (or more than 64): its KV heads, each cut into `splits` pieces.  A batch waits for its lengths here.  Cut
  // into as many pieces as there are sequences times splits, it deals them by length (deal_pieces), the KV heads of a
  // piece side by side (they read the same rows of the cache); uncut, the longest sequences go first.
  const bool batch = p.units_per_xcd > 0, dealt = batch && splits > 1;
  const int wid = (blockIdx.x & 7) * (p.total_wgs >> 3) + (blockIdx.x >> 3);
  const int rest = div_mg(wid, p.mg_qtiles), qtile = wid - rest * p.n_qtiles;
  int b, kv, split = 0, pieces = splits;  // the sequence, its KV head, which piece of how many
  int place0, place_step;                 // its pieces' places among all: place0 + s * place_step
  // Ordinary loads are issued by hand like the transfers behind them, and waited for by number: the compiler, which does
  // not know of the transfers, would wait for the oldest of its loads by waiting for all but a few of everything issued
  // since.
  constexpr int ROW_LOADS = kBlocks * DK + 2;
  int L_lane, L_one, L = p.max_prefix;
  auto bounded = [&](int len) { return len < 0 ? 0 : (len > p.max_prefix ? p.max_prefix : len); };
  const int n_ttiles = (T + kTileKeys - 1) / kTileKeys;
  if (batch) {
    const int order = div_mg(rest, p.mg_hkv);  // of the piece, or of the sequence
    kv = rest - order * p.Hkv;
    if (order >= p.B * splits) return;  // padding workgroup
    load_by_hand<kAskedLengths>(L_lane, p.prefix_len + min(lane, p.B - 1));  // (lane i: sequence i's)
    // (the page table's first 32 KB, a line a thread, on their way into the L2 while the pieces are dealt)
    int touched;
    const long long last = (long long)p.B * p.max_blocks - 1;
    load_by_hand<kAskedTable>(touched, PAGED ? p.block_table + (32 * tid < last ? 32 * tid : (int)last) : p.prefix_len);
    dev::wait_vm<1>();
    arrived<kAskedLengths>(L_lane);
    const int len = bounded(L_lane);
    if (dealt) {
      const Deal d = deal_pieces(lane < p.B ? (len + kTileKeys - 1) / kTileKeys + n_ttiles : 0, p.B, splits, lane);
      b = __popcll(__ballot(lane < p.B && d.first <= order)) - 1;
      split = order - __builtin_amdgcn_readlane(d.first, b);
      pieces = __builtin_amdgcn_readlane(d.pieces, b);
    } else {
      b = sequence_of_rank(len, p.B, order, lane);
    }
    dev::wait_vm<0>();
    dropped<kAskedTable>(touched);
    if (split >= pieces) return;  // (fewer pieces than places)
    L = __builtin_amdgcn_readlane(len, b);
    place0 = (order - split) * p.Hkv + kv;
    place_step = p.Hkv;
  } else {
    const int unit = div_mg(rest, p.mg_splits);
    if (unit >= p.B * p.Hkv) return;
    split = rest - unit * splits;
    b = div_mg(unit, p.mg_hkv);
    kv = unit - b * p.Hkv;
    place0 = unit * splits;
    place_step = 1;
    // (starts its K/V stream as if its prefix had the length of the bound, and again if it turns out shorter)
    load_by_hand<kAskedLength>(L_one, p.prefix_len + b);
  }
  // ---- the split's tiles
  TileSrc ts;
  ts.T = T;
  ts.kc_sl = p.kc_sl;
  ts.kt_st = p.kt_st;
  ts.pg_s = pg_s;
  ts.pg_first = 0;
  ts.tpp = p.tpp;
  ts.mg_tpp = p.mg_tpp;
  ts.page_stride = p.page_stride;
  auto set_range = [&](int len) {  // tiles dealt evenly, the longer shares first (the last piece has the masked ones)
    ts.L = len;
    ts.n_ptiles = (len + kTileKeys - 1) / kTileKeys;
    const int nt = ts.n_ptiles + n_ttiles, base = divided(nt, pieces), rem = nt - base * pieces;
    ts.t_begin = split * base + min(split, rem);
    ts.t_end = ts.t_begin + base + (split < rem ? 1 : 0);
  };
  set_range(L);
  int n = ts.t_end - ts.t_begin;
  bool bad_page = false;
  int n_pg = 0, first_id;  // pages of the list; this thread's first entry
  const int* table = p.block_table + (long long)b * p.max_blocks;
  auto ask_pages = [&]() {  // (see tva_bf16.hip)
    const int te = min(ts.n_ptiles, ts.t_end);
    n_pg = 0;
    if (te > ts.t_begin) {
      ts.pg_first = div_mg(ts.t_begin, p.mg_tpp);
      n_pg = div_mg(te - 1, p.mg_tpp) - ts.pg_first + 1;  // <= kMaxPagesPerSplit by the host's plan
    }
    // (a load by hand in every lane: the compiler may not move its result before it has been waited for)
    load_by_hand<kAskedPages>(first_id, tid < n_pg && ts.pg_first + tid < p.max_blocks ? table + ts.pg_first + tid : p.prefix_len);
  };
  auto fill_pages = [&]() {  // (the ids have been waited for)
    arrived<kAskedPages>(first_id);
    bad_page = false;
    for (int i = tid; i < n_pg && i < kMaxPagesPerSplit; i += kWideThreads) {
      const int pi = ts.pg_first + i;
      const int id = pi >= p.max_blocks ? 0 : (i == tid ? first_id : table[pi]);
      bad_page = bad_page || id < 0 || id >= p.n_pages;
      pg_s[i] = id < 0 ? 0 : (id >= p.n_pages ? p.n_pages - 1 : id);
    }
    __syncthreads();
  };
  // (the query rows come while the page ids do: behind them, and the transfers, they took 4.9 us of a call's first 10.8; what the
  // transfers need is worked out behind these requests)
  if (PAGED) ask_pages();
  __builtin_amdgcn_sched_barrier(0);
  const int row0 = qtile * QROWS + wave * kWideRows;  // the wave's first query row
  u32x4 q_raw[kBlocks][DK];
  int parent_lo, parent_hi;  // of nodes lane and lane + 64
#pragma unroll
  for (int r = 0; r < kBlocks; ++r) {
    const int mm = min(row0 + r * kWaveRows + c32, M - 1), node = div_mg(mm, p.mg_g);
    const uint16_t* src = p.q + (unsigned)b * (unsigned long long)p.q_sb + (unsigned)node * (unsigned long long)p.q_st +
                          (unsigned)(kv * G + (mm - node * G)) * (unsigned long long)p.q_sh + 8 * g;
    if (r == 0) load_rows_by_hand<kAskedRow>(q_raw[r], src);
    else load_rows_by_hand<kAskedRow + DK>(q_raw[r], src);
  }
  load_by_hand<kAskedParent>(parent_lo, p.parent + (long long)b * T + min(lane, T - 1));
  load_by_hand<kAskedParent + 1>(parent_hi, p.parent + (long long)b * T + min(lane + 64, T - 1));
  __builtin_amdgcn_sched_barrier(0);
  const unsigned ring_addr = (unsigned)(size_t)LDS_PTR(unsigned char, smem);
  LaneChunks<D, kWideWaves> lc;
  lane_chunks<D, kWideWaves>(lc, wave, lane, lane_column<D, kWideWaves>(wave, lane), ts);
  const bool is_v = wave * N >= G_::NB;
  lc.cache = uniform_ptr((is_v ? p.vc : p.kc) + (PAGED ? 0 : (unsigned)b * (unsigned long long)p.kc_sb) + (unsigned)kv * (unsigned long long)p.kc_sh);
  lc.tree = uniform_ptr((is_v ? p.vt : p.kt) + (unsigned)b * (unsigned long long)p.kt_sb + (unsigned)kv * (unsigned long long)p.kt_sh);
#pragma unroll
  for (int i = 0; i < N; ++i) lc.lds[i] = (wave * N) / G_::NB * P_::HALF_BYTES + (wave * N + i) % G_::NB * 1024;
  if (PAGED) {
    dev::wait_vm<ROW_LOADS>();
    fill_pages();
  }

  auto transfer = [&](int i) { dma_round<D, kWideWaves, 1, PAGED>(i, ts, lc, ring_addr + i % NR * TILE_BYTES); };
  const float inv_tpp = PAGED ? __builtin_amdgcn_rcpf((float)ts.tpp) : 0.f;
  auto first_transfers = [&]() {  // as many tiles as the ring takes, full prefix tiles in the shorter way
    const int most = min(n, (int)P_::AHEAD), full = min(ts.L / kTileKeys - ts.t_begin, most);
    const long long tile = (long long)kTileKeys * ts.kc_sl;
    PagedTile at;  // (lane i: tile i's)
    if (PAGED && full > 0) at = paged_tile(ts, min(lane, full - 1), inv_tpp);
    const uint16_t* base = lc.cache + (PAGED ? 0 : ts.t_begin * tile);
    int i = 0;
    for (; i < full; ++i) {
      const uint16_t* src = PAGED ? base + at.offset(i) : base;
#pragma unroll
      for (int c = 0; c < N; ++c) dma16(src, lc.off[c], ring_addr + i * TILE_BYTES + lc.lds[c]);
      if (!PAGED) base += tile;
    }
    for (; i < most; ++i) transfer(i);
  };
  first_transfers();
  if (!batch) {
    if (n >= P_::AHEAD) dev::wait_vm<ROW_LOADS + P_::AHEAD * N>();
    else dev::wait_vm<ROW_LOADS>();  // (no less than needed)
    L = bounded(__builtin_amdgcn_readfirstlane(taken<kAskedLength>(L_one)));
    if (L != p.max_prefix) {  // (uniform over the workgroup)
      dev::wait_vm<0>();  // the ring must be quiet before the same places are filled again
      __syncthreads();
      set_range(L);
      n = ts.t_end - ts.t_begin;
      if (PAGED) {
        ask_pages();
        dev::wait_vm<0>();
        fill_pages();
      }
      first_transfers();
    }
  }
  if (PAGED && bad_page) __hip_atomic_fetch_or(p.err, kDevErrBadPage, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (n >= P_::AHEAD) dev::wait_vm<P_::AHEAD * N>();
  else wait_dma<N>(n);
  arrived_rows<kAskedRow>(q_raw[0]);
  arrived_rows<kAskedRow + DK>(q_raw[1]);
  arrived<kAskedParent>(parent_lo);
  arrived<kAskedParent + 1>(parent_hi);
  dropped<kAskedLength>(L_one);
  if (lane >= T) parent_lo = -1;
  if (lane + 64 >= T) parent_hi = -1;
  // the sets are published by the barrier in front of the first tile
  if (ts.t_end > ts.n_ptiles && wave == 0) build_ancestor_sets(lane, T, parent_lo, parent_hi, par_s, anc);
  if (tid == 0) *repeat_s = 0;  // (read behind the barrier that follows the loop)

  WideState<D> st;
#pragma unroll
  for (int r = 0; r < kBlocks; ++r) {
    const bool ok = row0 + r * kWaveRows + c32 < M;
#pragma unroll
    for (int ks = 0; ks < DK; ++ks) {
      u32x4 v = q_raw[r][ks];
      if (!ok) v = u32x4{0u, 0u, 0u, 0u};
      st.q[r][ks] = __builtin_bit_cast(bf16x8, v);
      // (D = 128: in accumulation registers, from which only matrix instructions read it.  Left alone, the compiler moves
      // it between the two files in the tile loop.)
      if (D == 128) asm volatile("" : "+a"(st.q[r][ks]));
    }
  }
  // adds[i][k]: rows 4 G' ... of the result reach the lanes 16 G' ...; they add up the k groups (lanes 16 k' ... of the
  // weights) that hold the same query rows, i.e. those of equal parity
  {
    const bool one = (((lane >> 4) ^ (lane >> 2)) & 1) == 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) st.adds[e] = (__bf16)(one ? 1.f : 0.f);
  }
  auto clear = [&]() {
#pragma unroll
    for (int r = 0; r < kBlocks; ++r) {
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) st.o[r][db][i] = 0.f;
      st.l[r] = floatx4{0.f, 0.f, 0.f, 0.f};
      st.m[r] = -INFINITY;
      st.mu[r] = 0.f;
    }
  };
  clear();

  const unsigned k_lane = ring_addr + G_::k_lane(lane), v_lane = ring_addr + P_::HALF_BYTES + G_::v_lane(lane);
  auto k_read = [&](unsigned tile, int ks) { return lds_read128((k_lane ^ (ks << 5)) + tile); };
  auto v_read = [&](unsigned tile, int h) {
    return lds_read_tr2((v_lane ^ ((h % DB) << 6)) + tile + 16 * (h / DB) * G_::ROW_BYTES, 8 * G_::ROW_BYTES);
  };
  // The first tile and tiles with masks.  Hides the keys of tile t that rows must not see (those of a ragged prefix tile,
  // tree tiles) in block r's scores: a bit per key, spread over a register and used to choose between the score and -inf
  // (register i of a lane is key 8 * (i / 4) + 4 * g + i % 4 of the tile).  Then the rows' references: the largest score of
  // the first tile in which a row sees a key.  Weights 2^(s - m) may grow to 2^64 from there (bf16 and fp32 have the same
  // exponents): a larger one shows in the row's sum after the loop.  (No branches: a step is one run of code.)
  auto hide = [&](int t, int r) {
    const int tt = t - ts.n_ptiles, left = L - t * kTileKeys;
    const int node = div_mg(min(row0 + r * kWaveRows + c32, M - 1), p.mg_g);
    unsigned seen = reinterpret_cast<const unsigned*>(anc)[4 * node + (tt >= 0 ? tt : 0)];
    if (tt < 0) seen = left >= kTileKeys ? ~0u : (1u << left) - 1u;
    seen >>= 4 * g;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const unsigned keep = (unsigned)__builtin_amdgcn_sbfe((int)seen, 8 * (i / 4) + i % 4, 1);
      st.s[r][i] = __uint_as_float((__float_as_uint(st.s[r][i]) & keep) | (0xff800000u & ~keep));
    }
  };
  auto look = [&](int t, int r) {
    hide(t, r);
    const float tmax = half_swap_max(max16(st.s[r])) * scale_log2;
    st.m[r] = st.m[r] == -INFINITY ? tmax : st.m[r];
    st.mu[r] = st.m[r] == -INFINITY ? 0.f : st.m[r];
    // (no weights for rows past the end, which nobody stores: products with zeros take less power, and a long loop runs at the clock that
    // power allows.  16 sequences of 60 nodes, four heads to one: 16 of 256 rows; us, without / with: up to 4096 keys in pages 59.2 /
    // 58.3, with the pieces dealt faster, in one block 59.4 / 58.3; 8 of 4096 keys 50.9 / 50.5)
    if (row0 + r * kWaveRows + c32 >= M) st.mu[r] = 1e30f;
  };
  const int n_full = min(max(L / kTileKeys - ts.t_begin, 0), n);  // tiles without a mask, the split's first ones

  if (n > 0) {
    // ---- the tiles: the steps that walk_tiles puts in order (tva_wide_order.h)
    constexpr int HK = DK / 2;
    auto wait = [&](int left, auto most) {
      constexpr int MOST = decltype(most)::value;
      if (left >= MOST) dev::wait_vm<MOST * N>();
      else wait_dma<N>(left);  // (waits for more than it has to where more than six tiles may be left)
    };
    // where spare transfers go, and what they bring: the last tile without a mask once more
    const unsigned dump = ring_addr + P_::RING_BYTES + wave * (N * 1024);
    auto spare = [&]() {
      const uint16_t* src = prefix_tile_base<PAGED>(ts, lc.cache, ts.t_begin + n_full - 1);
#pragma unroll
      for (int c = 0; c < N; ++c) dma16(src, lc.off[c], dump + c * 1024);
    };
    // Tile 0: its scores for block 0; everything else of the pipeline starts with zeros
    auto first = [&]() {
#pragma unroll
      for (int ks = 0; ks < DK; ++ks) st.kf[ks] = k_read(0, ks);
      const floatx16 zero = {};
      const bf16x8 none = __builtin_bit_cast(bf16x8, u32x4{0u, 0u, 0u, 0u});
#pragma unroll
      for (int h = 0; h < 2 * DB; ++h) st.vf[h] = none;
      st.p[1][0] = st.p[1][1] = none;
      st.x[1] = zero;
#pragma unroll
      for (int e = 16 - 16 / (2 * DK); e < 16; ++e) st.x[1][e] = -INFINITY;  // (their exponentials are taken in A(0))
#pragma unroll
      for (int ks = 0; ks < DK; ++ks)
        st.s[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(st.kf[ks], st.q[0][ks], ks == 0 ? zero : st.s[0], 0, 0, 0);
    };
    // One tile, wherever it lies
    auto step = [&](int i) {
      const unsigned kt = (unsigned)((i + 1) % NR) * TILE_BYTES, vt = (unsigned)(i % NR) * TILE_BYTES;
      look(ts.t_begin + i, 0);
      phase<D, 1>(st, scale_log2, [&](int slot) {
        if (slot % 4 == 0) st.kf[slot / 4] = k_read(kt, slot / 4);
        if (slot % 4 == 2) st.vf[slot / 4] = v_read(vt, slot / 4);
      });
      look(ts.t_begin + i, 1);
      phase<D, 0>(st, scale_log2, [&](int slot) {
        if (slot < DK && slot % 2 == 0) st.kf[HK + slot / 2] = k_read(kt, HK + slot / 2);
        if (slot < DK && slot % 2 == 1) st.vf[HK + slot / 2] = v_read(vt, HK + slot / 2);
      });
    };
    // Four tiles without masks at a time, from tile 1 of the piece on: their places in the ring are known but for the
    // upper bits, and every LDS address is one of twelve registers and an immediate.  One run of code without branches:
    // its steps ask for full prefix tiles, or for the last of these once more where there is none left (to where
    // nobody reads it).
    unsigned here, there, ka[DK], va[DB];
    PagedTile at;
    const uint16_t* next;
    auto run = [&](int i) {
      here = (unsigned)((i - 1) % NR) * TILE_BYTES;
      there = (unsigned)((i + 3) % NR) * TILE_BYTES;
      unsigned kl = k_lane, vl = v_lane;
      asm volatile("" : "+v"(kl), "+v"(vl));  // (made anew: else twelve loop invariants, fetched from accumulation registers)
#pragma unroll
      for (int ks = 0; ks < DK; ++ks) {
        ka[ks] = (kl ^ (ks << 5)) + here;
        asm volatile("" : "+v"(ka[ks]));  // (held: else made anew at u == 2, out of accumulation registers, between matrix instructions)
      }
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        va[db] = (vl ^ (db << 6)) + here;
        asm volatile("" : "+v"(va[db]));
      }
      if (PAGED) at = paged_tile(ts, min(i + P_::AHEAD + (lane & 3), n_full - 1), inv_tpp);
      next = lc.cache + (PAGED ? 0 : (long long)(ts.t_begin + min(i + P_::AHEAD, n_full - 1)) * kTileKeys * ts.kc_sl);
    };
    auto run_step = [&](int i, int u) {
      const unsigned kt = (unsigned)((u + 2) % 4) * TILE_BYTES, vt = (unsigned)((u + 1) % 4) * TILE_BYTES;
      auto k_at = [&](int ks) { st.kf[ks] = lds_read128(ka[ks] + kt); };
      auto v_at = [&](int h) {
        st.vf[h] = lds_read_tr2(va[h % DB] + vt + 16 * (h / DB) * G_::ROW_BYTES, 8 * G_::ROW_BYTES);
      };
      phase<D, 1>(st, scale_log2, [&](int slot) {
        if (slot % 4 == 0) k_at(slot / 4);
        if (slot % 4 == 2) v_at(slot / 4);
      });
      const uint16_t* src = next;
      if (PAGED) src += at.offset(u);
      else next += i + u + P_::AHEAD < n_full - 1 ? (long long)kTileKeys * ts.kc_sl : 0;
      const unsigned to = i + u + P_::AHEAD < n_full ? ring_addr + lc.lds[0] + here + u * TILE_BYTES : dump;  // (the place of tile i + u - 1)
      phase<D, 0>(st, scale_log2, [&](int slot) {
        if (slot < DK && slot % 2 == 0) k_at(HK + slot / 2);
        if (slot < DK && slot % 2 == 1) v_at(HK + slot / 2);
#pragma unroll
        for (int c = 0; c < N; ++c)
          if (slot == DK + c * DK / N) dma16(src, lc.off[c], to + c * 1024);
      });
      // (for the next step, in front of its barrier)
      if (u == 1) {
#pragma unroll
        for (int ks = 0; ks < DK; ++ks) ka[ks] += there - here;
      }
      if (u == 2) {
#pragma unroll
        for (int db = 0; db < DB; ++db) va[db] += there - here;
      }
    };
    auto meet = [&]() {
      __syncthreads();
      // (a matrix instruction moved up in front of the barrier stalls the wave until the matrix unit takes it, and the
      // others wait for the wave: 1 % of a long call)
      __builtin_amdgcn_sched_barrier(0);
    };
    tva::walk_tiles<P_::AHEAD>(n, n_full, row0 >= M, transfer, spare, wait, meet, first, step, run, run_step);
    // ---- the last tile's value product for block 1
    softmax_rest<D, 1>(st, scale_log2);
#pragma unroll
    for (int h = 0; h < 2 * DB; ++h)
      st.o[1][h % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(st.vf[h], st.p[1][h / DB], st.o[1][h % DB], 0, 0, 0);
  }
  if (!(st.l[0][0] < 1.8446744e19f) || !(st.l[1][0] < 1.8446744e19f)) *repeat_s = 1;
  __syncthreads();  // everybody is done with the ring
  if (__builtin_amdgcn_readfirstlane(*repeat_s) != 0) {
    // ---- A weight beyond 2^64 (a score 44 nats above the row's first), or a sum that is no number: the split once
    // more, with a reference that moves and accumulators that follow it.  Rare, and in no hurry: one tile after the other.
    clear();
    for (int i = 0; i < n; ++i) {
      transfer(i);
      dev::wait_vm<0>();
      __syncthreads();
      const unsigned tile = (unsigned)(i % NR) * TILE_BYTES;
      const int t = ts.t_begin + i;
#pragma unroll
      for (int r = 0; r < kBlocks; ++r) {
        const floatx16 zero = {};
#pragma unroll
        for (int ks = 0; ks < DK; ++ks)
          st.s[r] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k_read(tile, ks), st.q[r][ks], ks == 0 ? zero : st.s[r], 0, 0, 0);
        if (i >= n_full) hide(t, r);
        const float tmax = half_swap_max(max16(st.s[r])) * scale_log2;
        const float m_new = fmaxf(st.m[r], tmax), mu = m_new == -INFINITY ? 0.f : m_new;
        const float alpha = fast_exp2(st.m[r] - mu);  // 0 before the first key: the accumulators are zero then
        st.m[r] = m_new;
        st.mu[r] = mu;
#pragma unroll
        for (int e = 0; e < 16; ++e) st.p[r][e / 8][e % 8] = (__bf16)fast_exp2(fmaf(st.s[r][e], scale_log2, -mu));
        // (added up without the matrix, whose zeros would carry a weight that is no number into the row 16 further)
        float sum = 0.f;
#pragma unroll
        for (int e = 0; e < 16; ++e) sum += (float)st.p[r][e / 8][e % 8];
        sum += __uint_as_float(dev::other32(__float_as_uint(sum), lane & 32));
#pragma unroll
        for (int k = 0; k < 4; ++k) st.l[r][k] = fmaf(st.l[r][k], alpha, sum);
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int k = 0; k < 16; ++k) st.o[r][db][k] *= alpha;
#pragma unroll
        for (int h = 0; h < 2 * DB; ++h)
          st.o[r][h % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v_read(tile, h), st.p[r][h / DB], st.o[r][h % DB], 0, 0, 0);
      }
    }
    __syncthreads();
  }

  // ---- Merge of the pieces, two and two: the steps of merge_pieces (tva_wide_order.h).  Results are left in fp32 and in the
  // order of the registers.  The sum is the same whoever comes first.  The two may run on different XCDs, whose L2s know
  // nothing of each other: stores go through to memory, and the loads bypass them (sc1, the scope of the device).
  constexpr int QUADS = kBlocks * DB * 4;  // float4 per lane
  constexpr int kDeviceScope = 16;         // (the sc1 bit of a buffer load)
  auto place_of = [&](int piece) { return (place0 + piece * place_step) * p.n_qtiles + qtile; };
  auto word_of = [&](int m) { return p.sync + wide_word(place_of(m)); };
  int* answer_s = repeat_s + 1;  // thread 0's answer; two in turn, so that one barrier does
  bool is_first = false;         // (thread 0's)
  auto answered = [&]() {
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(*answer_s);
  };
  auto arrive = [&](int m) {
    answer_s = repeat_s + (answer_s == repeat_s + 1 ? 2 : 1);
    if (tid == 0) {
      unsigned* word = word_of(m);
      unsigned was = __hip_atomic_fetch_add(word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      is_first = was == 0u;
      int at = -1;
      if (!is_first) {  // (the other workgroup has come: it has nothing left to do but its stores)
        unsigned polls = 0;
        for (;;) {
          at = tva::others_results(was, false);  // (usually in what the addition found: no trip more)
          if (at >= 0) break;
          if (++polls > p.spin_limit) {
            __hip_atomic_fetch_or(p.err, kDevErrMergeWait, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            break;
          }
          __builtin_amdgcn_s_sleep(1);
          was = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
      *answer_s = at;
    }
    return answered();
  };
  auto leave = [&](int m) {
    const int place = place_of(split);
    if (row0 < M) {
      float4* part = reinterpret_cast<float4*>(p.part_o) + (size_t)(place * kWideWaves + wave) * (QUADS * 64) + lane;
      float2* ml = p.part_ml + (size_t)place * QROWS + wave * kWideRows + c32;
#pragma unroll
      for (int r = 0; r < kBlocks; ++r) {
        dev::store_through(ml + r * kWaveRows, dev::store_u32x2{__float_as_uint(st.m[r]), __float_as_uint(st.l[r][0])});
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) {
            const floatx16& o = st.o[r][db];
            dev::store_through(part + ((r * DB + db) * 4 + q4) * 64,
                               dev::store_u32x4{__float_as_uint(o[4 * q4]), __float_as_uint(o[4 * q4 + 1]), __float_as_uint(o[4 * q4 + 2]), __float_as_uint(o[4 * q4 + 3])});
          }
      }
    }
    dev::wait_vm<0>();
    __syncthreads();
    if (tid == 0)
      *answer_s = tva::others_results(__hip_atomic_fetch_or(word_of(m), tva::left_results(is_first, split), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), is_first);
    return answered();
  };
  auto add = [&](int m, int at) {
    if (tid == 0) __hip_atomic_store(word_of(m), 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (row0 >= M) return;
    const int place = place_of(at);
    const float2* ml = p.part_ml + (size_t)place * QROWS + wave * kWideRows + c32;
    const auto theirs = __builtin_amdgcn_make_buffer_rsrc(p.part_o + (size_t)(place * kWideWaves + wave) * (QUADS * 64 * 4), 0, QUADS * 64 * 16, 0x00020000);
#pragma unroll
    for (int r = 0; r < kBlocks; ++r) {
      const u32x2 other = __builtin_bit_cast(u32x2, __hip_atomic_load(reinterpret_cast<const uint64_t*>(ml + r * kWaveRows), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
      const float other_m = __uint_as_float(other[0]), other_l = __uint_as_float(other[1]);
      u32x4 v[DB * 4];  // (all on their way before the first is used)
#pragma unroll
      for (int i = 0; i < DB * 4; ++i) v[i] = __builtin_amdgcn_raw_buffer_load_b128(theirs, lane * 16, (r * DB * 4 + i) * 1024, kDeviceScope);
      __builtin_amdgcn_sched_barrier(0);
      const float m_new = fmaxf(st.m[r], other_m), mu = m_new == -INFINITY ? 0.f : m_new;
      const float w0 = fast_exp2(st.m[r] - mu), w1 = fast_exp2(other_m - mu);  // (exp2(-inf) = 0: a row without a key)
      st.m[r] = m_new;
      // (no fused multiply-add: it would round one of the two products only, and which one would be up to who came first)
      auto sum = [&](float x, float y) {
#pragma clang fp contract(off)
        const float a = x * w0, c = y * w1;
        return a + c;
      };
      st.l[r][0] = sum(st.l[r][0], other_l);
#pragma unroll
      for (int i = 0; i < DB * 4; ++i) {
        floatx16& o = st.o[r][i / 4];
#pragma unroll
        for (int k = 0; k < 4; ++k) o[4 * (i % 4) + k] = sum(o[4 * (i % 4) + k], __uint_as_float(v[i][k]));
      }
    }
  };
  if (!tva::merge_pieces(split, pieces, arrive, leave, add)) return;

  // ---- the finished rows, a block of 32 at a time through a patch of LDS so that they leave in whole 128-byte lines (see
  // tva_bf16.hip)
  const bool thr = (p.through & 1) != 0;
  constexpr int CPR = G_::CPR, RPI = 64 / CPR;
  const int chunk = lane % CPR, rsub = lane / CPR;
  unsigned char* patch = smem + wave * P_::PATCH_BYTES;
  unsigned char* prow = patch + c32 * P_::PATCH_LD;
  const unsigned char* src0 = patch + rsub * P_::PATCH_LD + chunk * 16;
  uint16_t* out0 = p.out + b * p.o_sb + (long long)kv * G * p.o_sh + chunk * 8;
#pragma unroll
  for (int r = 0; r < kBlocks; ++r) {
    const int first = row0 + r * kWaveRows, rows_valid = M - first;
    if (rows_valid <= 0) break;
    const float mul = 1.f / st.l[r][0];  // > 0: every row sees at least its own tree key
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        bf16x2 lo, hi;
        lo[0] = (__bf16)(st.o[r][db][4 * q4] * mul);
        lo[1] = (__bf16)(st.o[r][db][4 * q4 + 1] * mul);
        hi[0] = (__bf16)(st.o[r][db][4 * q4 + 2] * mul);
        hi[1] = (__bf16)(st.o[r][db][4 * q4 + 3] * mul);
        uint2 pk;
        pk.x = __builtin_bit_cast(unsigned int, lo);
        pk.y = __builtin_bit_cast(unsigned int, hi);
        *reinterpret_cast<uint2*>(prow + (32 * db + 8 * q4 + 4 * g) * 2) = pk;
      }
    // (same wave wrote and reads: LDS operations of a wave complete in order)
    auto store_rows = [&](auto through) {
#pragma unroll
      for (int k = 0; k < kWaveRows / RPI; ++k) {
        const u32x4 v = *reinterpret_cast<const u32x4*>(src0 + k * RPI * P_::PATCH_LD);
        const int m = first + k * RPI + rsub, node = div_mg(m, p.mg_g);
        uint16_t* dst = out0 + node * p.o_st + (long long)(m - node * G) * p.o_sh;
        if (m >= M) continue;
        if (decltype(through)::value) dev::store_through(dst, v);
        else *reinterpret_cast<u32x4*>(dst) = v;
      }
    };
    if (thr) store_rows(std::true_type{});
    else store_rows(std::false_type{});
  }
}

template <int D, bool PAGED>
hipError_t launch_one(const KParams& kp, hipStream_t stream) {
  using P_ = WidePlan<D, PAGED>;
  auto kern = tva_wide_kernel<D, PAGED>;
  static LdsLimitRaised raised;
  if (hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(kern), P_::SMEM, raised); e != hipSuccess) return e;
  return launch_kernel(kern, dim3(kp.total_wgs), dim3(kWideThreads), P_::SMEM, stream, kp);
}

}  // namespace

namespace tva {
hipError_t launch_wide(const KParams& kp, int head_dim, hipStream_t stream) {
  const bool paged = kp.block_table != nullptr;
  if (head_dim == 128) return paged ? launch_one<128, true>(kp, stream) : launch_one<128, false>(kp, stream);
  if (head_dim == 64) return paged ? launch_one<64, true>(kp, stream) : launch_one<64, false>(kp, stream);
  return hipErrorInvalidValue;
}
}  // namespace tva

}  // namespace jk
