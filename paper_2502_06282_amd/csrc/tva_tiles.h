// What the bf16 tree-attention kernels share (tva_bf16.hip, tva_wide.hip): their parameters, the swizzled layout of a 32-key
// K/V tile in LDS, the transfers that fill it and the masks.  Not installed.
#pragma once
#include "jk_device.h"
#include "jk_internal.h"

namespace jk {
namespace tva {
struct KParams {
  const uint16_t *q, *kc, *vc, *kt, *vt;
  const int32_t *parent, *prefix_len;
  uint16_t* out;
  float* part_o;
  float2* part_ml;
  int B, T, Hkv, G, M, m_pad, max_prefix, splits, n_qtiles, total_wgs;
  unsigned long long mg_qtiles, mg_splits, mg_hkv, mg_g;  // floor(2^32 / d) + 1: n / d == (n * mg) >> 32 for n * d < 2^32
  unsigned long long mg_splits_m1;                        // the same for max(splits - 1, 1)
  long long q_sb, q_st, q_sh, kc_sb, kc_sl, kc_sh, kt_sb, kt_st, kt_sh, o_sb, o_st, o_sh;
  float scale_log2;
  // paged cache (block_table != nullptr): kc / vc are page pools, token t of sequence b lives in page
  // block_table[b * max_blocks + t / page_size], slot t % page_size; tpp = 32-key tiles per page
  const int32_t* block_table;
  int max_blocks, tpp, n_pages;
  int through;  // bit 0: outputs and partials, bit 1: the partials' (max, sum) pairs go through to memory; bit 2: the partials
                // are fp32 (see the epilogue)
  long long page_stride;
  unsigned long long mg_tpp;
  // split merge inside this kernel (MERGE > 0; see merge_rows and the end of the kernel): sync = one
  // 64-byte line of words per (unit, row tile) group in the workspace header, spin_limit = polls a
  // workgroup spends waiting for its group before it leaves its slice to the group's last arriver
  // (tva_wide.hip: for another one's stores, before it leaves its results too)
  unsigned* sync;
  unsigned* err;  // the workspace's sticky device error word
  unsigned spin_limit;
  int merge_rows, merge_shift;  // rows per slice = ceil(tile rows / splits); splits padded to 2^merge_shift
  // batches: the sequences by falling length, dealt to the XCDs in turn (units_per_xcd > 0; see the kernel's start)
  int units_per_xcd, second_turn;
  unsigned long long mg_upx;
};

// One call with the kernel of 256 query rows per workgroup (tva_wide.hip)
hipError_t launch_wide(const KParams& kp, int head_dim, hipStream_t stream);
// One undivided call with the kernel of 16 query rows per workgroup that takes K and V straight into registers (tva_direct.hip)
hipError_t launch_direct(const KParams& kp, int head_dim, hipStream_t stream);
}  // namespace tva

namespace {
using tva::KParams;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef short shortx8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));  // native vector: plain loads/stores, no struct copies
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

#define LDS_PTR(T, p) ((__attribute__((address_space(3))) T*)(p))

typedef __attribute__((address_space(3))) const bf16x8 lds_bf16x8;
typedef __attribute__((address_space(3))) shortx4 lds_shortx4;

// LDS reads by byte address.  Tile bases are multiples of 256 bytes, so the XOR swizzles can
// be applied to the finished address: one address register per operand stream plus an
// immediate per read, instead of a register per read.
__device__ __forceinline__ bf16x8 lds_read128(unsigned addr) { return *(lds_bf16x8*)(size_t)addr; }
__device__ __forceinline__ bf16x8 lds_read_tr2(unsigned addr, unsigned second) {
  const shortx4 x0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4*)(size_t)addr);
  const shortx4 x1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4*)(size_t)(addr + second));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(x0, x1, 0, 1, 2, 3, 4, 5, 6, 7));
}

constexpr int kWaveRows = 32;   // query rows per wave
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// n / d by multiplication with the host-made constant mg = floor(2^32 / d) + 1 (exact while n * d < 2^32)
__device__ __forceinline__ int div_mg(int n, unsigned long long mg) {
  return (int)(((unsigned long long)(unsigned)n * mg) >> 32);
}

// max over the two half-waves (lane l and lane l^32)
__device__ __forceinline__ float half_swap_max(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float half_swap_sum(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

template <int D>
struct Geo {
  static constexpr int ROW_BYTES = D * 2;
  static constexpr int TILE_BYTES = kTileKeys * ROW_BYTES;
  static constexpr int CPR = D / 8;               // 16-byte chunks per row
  static constexpr int DK = D / 16;               // k-steps of Q.K^T
  static constexpr int DB = D / 32;               // 32-wide d blocks of the output
  static constexpr int NB = TILE_BYTES / 1024;    // 1 KB transfers per tile and tensor
  __device__ static __forceinline__ int kswz(int row) { return (row / (16 / CPR)) % CPR; }
  __device__ static __forceinline__ int vswz(int row) { return (row / (4 / DB)) % DB; }
  // K operand of k-step ks (A of S^T = K . Q^T; lane = key row c32, half g): chunk
  // (2*ks + g) ^ kswz of its row = byte address (tile + k_lane(lane)) ^ (ks << 5)
  __device__ static __forceinline__ unsigned k_lane(int lane) {
    const int c32 = lane & 31, g = lane >> 5;
    return (unsigned)(c32 * ROW_BYTES + ((kswz(c32) ^ g) << 4));
  }
  // V^T operand (transpose read: the 16 lanes of a group address 4 keys x 32 bytes, lane i of
  // the group receives d-column i of those 4 keys; contraction index 4*q'+r of MFMA j is key
  // 16*j + 8*q' + 4*g + r): 64-byte block db ^ vswz of key row 4*g + (lane%16)/4 = byte
  // address ((tile + v_lane(lane)) ^ (db << 6)) + 16*j*ROW_BYTES, second half 8 rows further
  __device__ static __forceinline__ unsigned v_lane(int lane) {
    const int g = lane >> 5, jj = (lane & 15) >> 2, cc = lane & 3, h16 = (lane & 31) >> 4;
    const int key_lo = 4 * g + jj;
    return (unsigned)(key_lo * ROW_BYTES + 32 * h16 + 8 * cc + (vswz(key_lo) << 6));
  }
};

// Ordinary loads by hand (what waits for them says how many transfers may have been issued since).  The compiler takes their results to be
// there at once.  So until the wait a result's register must be neither moved nor given to another value: every path that asks for one
// gets to an arrived(), taken() or dropped() of it behind the wait, whether the value is of use there or not.  TAG names the value in the listing, where a
// test compares the registers of both.
enum Asked { kAskedLengths, kAskedLength, kAskedPages, kAskedTable, kAskedPair, kAskedParent, kAskedRow = 8 };  // (parents: two; rows: up to sixteen)
template <int TAG>
__device__ __forceinline__ void load_by_hand(int& v, const void* src) {
  asm volatile("global_load_dword %0, %1, off ; asked %0 as %2" : "=v"(v) : "v"(src), "n"(TAG) : "memory");
}
// N times 16 bytes, every 32 bytes
template <int TAG, int N, int I = 0>
__device__ __forceinline__ void load_rows_by_hand(u32x4 (&v)[N], const void* src) {
  if constexpr (I < N) {
    asm volatile("global_load_dwordx4 %0, %1, off offset:%2 ; asked %0 as %3" : "=v"(v[I]) : "v"(src), "n"(32 * I), "n"(TAG + I) : "memory");
    load_rows_by_hand<TAG, N, I + 1>(v, src);
  }
}
// Behind the wait, and in front of every use
template <int TAG, class T>
__device__ __forceinline__ void arrived(T& v) {
  asm volatile("; arrived %0 as %1" : "+v"(v) : "n"(TAG));
}
template <int TAG, int N, int I = 0>
__device__ __forceinline__ void arrived_rows(u32x4 (&v)[N]) {
  if constexpr (I < N) {
    arrived<TAG + I>(v[I]);
    arrived_rows<TAG, N, I + 1>(v);
  }
}
template <int TAG>
__device__ __forceinline__ void dropped(const int& v) {  // (as arrived(), where no use comes any more)
  asm volatile("; arrived %0 as %1" ::"v"(v), "n"(TAG));
}
// A copy, where several paths have a use of their own: with arrived() in each, the compiler would move the value in front of them
template <int TAG>
__device__ __forceinline__ int taken(const int& v) {
  int copy;
  asm volatile("v_mov_b32 %0, %1 ; arrived %1 as %2" : "=v"(copy) : "v"(v), "n"(TAG));
  return copy;
}

using dev::dma16;
using dev::uniform_ptr;

// Wait until at most `rounds_behind` rounds of this wave's transfers are still in flight
// (they complete in issue order).  The count must be an immediate, hence the switch.
template <int STEP>
__device__ __forceinline__ void wait_dma(int rounds_behind) {
#define JK_VM(n) __builtin_amdgcn_s_waitcnt(dev::vmcnt_imm(n))
  switch (rounds_behind) {
    case 0: JK_VM(0); break;
    case 1: JK_VM(STEP); break;
    case 2: JK_VM(2 * STEP); break;
    case 3: JK_VM(3 * STEP); break;
    case 4: JK_VM(4 * STEP); break;
    case 5: JK_VM(5 * STEP); break;
    default: JK_VM(6 * STEP); break;
  }
#undef JK_VM
}

// The K/V streams of this (sequence, KV head) and the tile range of this split.
struct TileSrc {
  long long kc_sl, kt_st;  // row strides (elements)
  int L, T, n_ptiles, t_begin, t_end;
  // paged cache: page ids of the split's prefix tiles (LDS), index of the first one, tiles per page
  const int* pg_s;
  int pg_first, tpp;
  unsigned long long mg_tpp;
  long long page_stride;
};

constexpr int kMaxPagesPerSplit = 1024;  // page ids a workgroup keeps in LDS (the host keeps splits within it)

// Where a lane's 16-byte chunks sit inside a tile.  A wave-level transfer fills 1 KB =
// 64/CPR consecutive tile rows; lane l writes physical chunk l%CPR of row blk*(64/CPR) +
// l/CPR and fetches the logical chunk that the swizzle maps there, so the tile arrives
// already swizzled.  The 2*NB transfers of a tile (NB for K, then NB for V) are dealt to
// the NW waves in order, N to each: a wave therefore fetches only K or only V chunks.
template <int D, int NW>
struct LaneChunks {
  static constexpr int N = 2 * Geo<D>::NB / NW;
  static_assert(N >= 1 && Geo<D>::NB % N == 0, "a wave's transfers stay within K or within V");
  unsigned off[N];        // byte offset of the chunk from the first row of a full cache tile
  unsigned lds[N];        // byte offset inside the K+V tile pair
  const uint16_t* cache;  // K or V cache of this (sequence, KV head), wave-uniform
  const uint16_t* tree;   // K or V of the tree
  int wave, lane;
  // tile row and byte offset inside the row of chunk i: recomputed where the rare clamped
  // transfers need them rather than held in registers across the tile loop
  __device__ __forceinline__ void where(int i, int& row, unsigned& col_b) const {
    using G_ = Geo<D>;
    constexpr int RPB = 64 / G_::CPR;
    const int is_v = (wave * N) / G_::NB;
    const int blk = (wave * N + i) % G_::NB;
    row = blk * RPB + lane / G_::CPR;
    const int pc = lane % G_::CPR;
    const int kcol = pc ^ G_::kswz(row);                                  // K: 16-byte chunks swizzled
    const int vcol = (((pc >> 2) ^ G_::vswz(row)) << 2) | (pc & 3);       // V: 64-byte blocks swizzled
    col_b = (unsigned)(is_v ? vcol : kcol) * 16u;
  }
};

// The part of a chunk's byte offset in its row that does not depend on which of the wave's chunks it is.  A wave's rows are a
// multiple of 64 / CPR apart, so `where`'s swizzles come apart: V's is the same for all of them, K's differs by a
// constant in the bits above.
template <int D, int NW>
__device__ __forceinline__ unsigned lane_column(int wave, int lane) {
  using G_ = Geo<D>;
  const int lr = lane / G_::CPR, pc = lane % G_::CPR;
  const int k_swz = lr / (16 / G_::CPR), v_swz = lr / (4 / G_::DB) % G_::DB << 2;
  return (unsigned)(pc ^ (wave * LaneChunks<D, NW>::N >= G_::NB ? v_swz : k_swz)) * 16u;
}
// `column`: lane_column's, worked out while the kernel's arguments are on their way
template <int D, int NW>
__device__ __forceinline__ void lane_chunks(LaneChunks<D, NW>& lc, int wave, int lane, unsigned column, const TileSrc& ts) {
  using G_ = Geo<D>;
  constexpr int N = LaneChunks<D, NW>::N, RPB = 64 / G_::CPR;
  const bool is_v = wave * N >= G_::NB;
  lc.wave = wave;
  lc.lane = lane;
  const unsigned row_bytes = (unsigned)ts.kc_sl * 2u;  // < 2^25: strides are bounded by the host
  unsigned lane_rows = (unsigned)(lane / G_::CPR) * row_bytes;
  asm("" : "+v"(lane_rows));  // (one product, not one a chunk)
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const unsigned blk = (unsigned)(wave * N % G_::NB + i), k_swz = is_v ? 0u : blk % (unsigned)(G_::CPR / 4) * 64u;
    lc.off[i] = (column ^ k_swz) + (lane_rows + blk * (unsigned)RPB * row_bytes);
    lc.lds[i] = (is_v ? G_::TILE_BYTES : 0) + blk * 1024;
  }
}

// First row of prefix tile t of this (sequence, KV head): contiguous cache, or looked up in the
// split's page list (the tile never straddles pages: a page holds whole tiles).
template <bool PAGED>
__device__ __forceinline__ const uint16_t* prefix_tile_base(const TileSrc& ts, const uint16_t* cache, int t) {
  if (!PAGED) return cache + (long long)t * kTileKeys * ts.kc_sl;
  const int pi = div_mg(t, ts.mg_tpp);
  const int page = __builtin_amdgcn_readfirstlane(ts.pg_s[pi - ts.pg_first]);
  return cache + (long long)page * ts.page_stride + (long long)(t - pi * ts.tpp) * kTileKeys * ts.kc_sl;
}

// Lane i < batch (at most 64) brings sequence i's length (at most 2^24): the sequence that `rank` others go in front of,
// longer ones and equal ones of a lower number.
__device__ __forceinline__ int sequence_of_rank(int len, int batch, int rank, int lane) {
  const int key = lane < batch ? (len << 6) | (63 - lane) : -1;  // (all different: one comparison each)
  int in_front = 0;
  for (int i = 0; i < batch; i += 4)  // (what lies past the batch's end goes in front of nobody)
#pragma unroll
    for (int k = 0; k < 4; ++k) in_front += (int)(__builtin_amdgcn_readlane(key, i + k) > key);
  return __ffsll((long long)__ballot(lane < batch && in_front == rank)) - 1;
}

// Issue the transfers of round r (TPR tiles, K and V) into ring slot `slot` (byte address).
template <int D, int NW, int TPR, bool PAGED>
__device__ __forceinline__ void dma_round(int r, const TileSrc& ts, const LaneChunks<D, NW>& lc, unsigned slot) {
  using G_ = Geo<D>;
  constexpr int N = LaneChunks<D, NW>::N;
  const int t0 = ts.t_begin + r * TPR;
  if ((t0 + TPR) * kTileKeys <= ts.L) {
    // every tile of the round is a full prefix tile: a scalar base per tile plus the lane's
    // precomputed offsets
    if (!PAGED) {
      const long long tile_elems = (long long)kTileKeys * ts.kc_sl;
      const uint16_t* base = lc.cache + (long long)t0 * tile_elems;
#pragma unroll
      for (int w = 0; w < TPR; ++w) {
#pragma unroll
        for (int i = 0; i < N; ++i) dma16(base, lc.off[i], slot + w * 2 * G_::TILE_BYTES + lc.lds[i]);
        base += tile_elems;
      }
    } else {
#pragma unroll
      for (int w = 0; w < TPR; ++w) {
        const uint16_t* base = prefix_tile_base<true>(ts, lc.cache, t0 + w);
#pragma unroll
        for (int i = 0; i < N; ++i) dma16(base, lc.off[i], slot + w * 2 * G_::TILE_BYTES + lc.lds[i]);
      }
    }
    return;
  }
#pragma unroll 1
  for (int w = 0; w < TPR; ++w) {
    int t = t0 + w;
    if (t >= ts.t_end) t = ts.t_end - 1;  // duplicate of a real tile, never consumed
    const unsigned dst = slot + w * 2 * G_::TILE_BYTES;
    // ragged last prefix tile or tree tile: rows past the end re-read the last valid row
    const bool tree = t >= ts.n_ptiles;
    const int key0 = (tree ? t - ts.n_ptiles : t) * kTileKeys;
    const int last = (tree ? ts.T : ts.L) - 1 - key0;  // >= 0 (and >= 31 for a full prefix tile)
    const long long rs = tree ? ts.kt_st : ts.kc_sl;
    const uint16_t* base = tree ? lc.tree + (long long)key0 * rs : prefix_tile_base<PAGED>(ts, lc.cache, t);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      int row;
      unsigned col_b;
      lc.where(i, row, col_b);
      const int rr = row < last ? row : last;
      dma16(base, (unsigned)rr * (unsigned)rs * 2u + col_b, dst + lc.lds[i]);
    }
  }
}

// Largest of a lane's 16 scores of a tile, as a tree three levels deep: a chain of fifteen
// dependent maxima would spend its latency with nothing else to issue.
__device__ __forceinline__ float max16(const floatx16& s) {
  const float a = fmaxf(fmaxf(s[0], s[1]), s[2]), b = fmaxf(fmaxf(s[3], s[4]), s[5]);
  const float c = fmaxf(fmaxf(s[6], s[7]), s[8]), d = fmaxf(fmaxf(s[9], s[10]), s[11]);
  const float e = fmaxf(fmaxf(s[12], s[13]), s[14]);
  return fmaxf(fmaxf(fmaxf(a, b), c), fmaxf(fmaxf(d, e), s[15]));
}

// Hide the masked keys of one tile's scores.  mask_mode: 0 none, 1 ragged prefix tail (keys
// >= nvalid hidden), 2 tree tile (bits = visibility of the tile's 32 keys; 0 for a tile
// past the end of the split).  Register i of a lane is key 8*(i/4) + 4*g + i%4 of the tile.
__device__ __forceinline__ void mask_tile(floatx16& sacc, int mask_mode, int nvalid, unsigned int bits, int g) {
  if (mask_mode == 0) return;
  // masked tiles are rare: keep their per-register key indices out of the loop-invariant
  // registers (the compiler would otherwise hold 32 of them across the whole tile loop)
  asm volatile("" : "+v"(g));
  if (mask_mode == 2) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int kk = 8 * (i / 4) + 4 * g + (i % 4);
      if (!((bits >> kk) & 1u)) sacc[i] = -INFINITY;
    }
  } else if (mask_mode == 1) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int kk = 8 * (i / 4) + 4 * g + (i % 4);
      if (kk >= nvalid) sacc[i] = -INFINITY;
    }
  }
}

// Ancestor sets of a tree's nodes (128 bits each), by pointer
// doubling: after k steps a node knows its nearest 2^k ancestors-or-self and its 2^k-th
// ancestor, so the number of steps is logarithmic in the depth of the tree rather than
// the depth itself (every step is a round trip through LDS).  One wave does it alone, two
// nodes per lane (parents of nodes lane and lane + 64): the LDS operations of a wave complete in program order, so the steps
// need no barrier (as rounds of the whole workgroup, with two or three barriers each, the
// same steps took three times as long, and the split that owns the tree tiles is the one
// the others wait for).  PARAMS_AT: where the kernel's KParams lie among its arguments.
template <int PARAMS_AT = 0>
__device__ __forceinline__ void build_ancestor_sets(int lane, int T, int parent_lo, int parent_hi, int* par_s,
                                                    unsigned long long* anc) {
  const int n_lo = lane, n_hi = lane + 64;
  int up_lo = (parent_lo >= -1 && parent_lo < n_lo) ? parent_lo : -1;  // indices strictly decrease towards the root
  int up_hi = (parent_hi >= -1 && parent_hi < n_hi) ? parent_hi : -1;  // (-1 as well for lanes past the tree)
  // an entry that breaks -1 <= parent[i] < i was just replaced by -1: say so in the workspace's error word
  if (up_lo != parent_lo || up_hi != parent_hi) {
    typedef __attribute__((address_space(4))) const KParams KArgs;
    KArgs* late = (KArgs*)((__attribute__((address_space(4))) const char*)__builtin_amdgcn_kernarg_segment_ptr() + PARAMS_AT);
    asm volatile("" : "+s"(late));  // (fetched here: not worth a scalar register pair across the kernel)
    __hip_atomic_fetch_or(late->err, kDevErrBadTree, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  unsigned long long lo_lo = n_lo < T ? 1ull << n_lo : 0ull, hi_lo = 0ull;  // node lane: bit < 64
  unsigned long long lo_hi = 0ull, hi_hi = n_hi < T ? 1ull << lane : 0ull;  // node lane + 64: bit >= 64
  const bool two = T > 64;  // uniform
  for (;;) {
    par_s[n_lo] = up_lo;
    anc[2 * n_lo] = lo_lo;
    anc[2 * n_lo + 1] = hi_lo;
    if (two) {
      par_s[n_hi] = up_hi;
      anc[2 * n_hi] = lo_hi;
      anc[2 * n_hi + 1] = hi_hi;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (!__any(up_lo >= 0 || up_hi >= 0)) break;  // nobody has an ancestor left to fold in: LDS holds the sets
    if (up_lo >= 0) {
      lo_lo |= anc[2 * up_lo];
      hi_lo |= anc[2 * up_lo + 1];
      up_lo = par_s[up_lo];
    }
    if (two && up_hi >= 0) {
      lo_hi |= anc[2 * up_hi];
      hi_hi |= anc[2 * up_hi + 1];
      up_hi = par_s[up_hi];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // every read of this step precedes the next step's writes
    __builtin_amdgcn_wave_barrier();
  }
}

}  // namespace
}  // namespace jk
