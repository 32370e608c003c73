// Tree-masked verification attention, bf16 inputs, MFMA path (gfx950).
//
// What it computes (Section 2.1 step 2 of the paper: the target model scores
// all draft candidates in one pass; Section 3.1.2: candidates form a tree and
// are verified through a tree attention mask): every tree node attends to the
// committed KV prefix, to itself and to its tree ancestors.
//
// Mapping.  The G query heads that share one KV head and the T tree nodes are
// packed into one matrix of M = T*G query rows (row m = node m/G, head m%G), so
// a KV head's K/V stream is read once for all of them.  One workgroup of
// WM x WN waves owns 32*WM query rows of one (sequence, KV head) and one split
// of the key range; the key range (prefix tiles, then tree tiles, 32 keys each)
// is cut into `splits` contiguous pieces.  Wave (wm, wn) holds query rows
// [32*wm, 32*wm+32) and processes every WN-th tile.  Workgroups have 4 waves
// (4x1 or 2x2) and two of them fit a CU: a single wave per SIMD is bound by its
// own in-order instruction issue (MFMA chain, exponentials, transfer
// bookkeeping), which a second workgroup on the CU overlaps.  (8-wave 2x4
// workgroups measured no better: they start later and their wider epilogue
// merge costs what the shorter tile loop gains.)
//
// Per tile and wave, with everything transposed so that a lane owns one query
// row:   S^T = K . Q^T   (v_mfma_f32_32x32x16_bf16, A = K rows from LDS,
// B = Q rows held in registers), masking, online softmax (running max and sum,
// max exchanged between the two half-waves with v_permlane32_swap), then
// O^T += V^T . P^T with V^T operands fetched by LDS transpose reads
// (ds_read_b64_tr_b16) from the row-major V tile.  The tree mask is a 128-bit
// ancestor set per node, built in LDS by the workgroups that own tree tiles.
//
// K/V travel HBM -> LDS directly (global_load_lds_dwordx4: 16 bytes per lane,
// 16 lanes per 256-byte row) into a ring of tiles, rounds ahead in flight;
// each lane fetches the 16-byte chunk that the XOR swizzle maps to its LDS
// slot, so that both the 128-bit K reads and the transpose V reads are free of
// bank conflicts.
#include <type_traits>

#include "tva_tiles.h"

// This file is compiled once for each way of merging the splits (JK_MERGE = 0 - 6, see merge_of): the instances build
// side by side.  The host's part is in the first.
#ifndef JK_MERGE
#error "compile with -DJK_MERGE=0 ... 6"
#endif

namespace jk {
namespace tva {
// How a kernel merges its splits (MERGE): 0 not at all (one split, or a second launch), then
//   1 two splits, 2 three: fp32 partials (see AttnPlan::fine)    3 four, 4 up to eight, 5 up to sixteen, 6 more: bf16
constexpr int merge_of(int splits) {
  return splits <= 4 ? splits - 1 : splits <= 8 ? 4 : splits <= 16 ? 5 : 6;
}
// 2^shift splits go through merge_rows at once (6: sixteen of more)
constexpr int merge_shift_of(int merge) { return merge <= 2 ? merge : merge - 1; }

// One call, merged as MERGE says, with the kernel for its head_dim and wave arrangement
template <int MERGE>
hipError_t launch_merged(const KParams& kp, int head_dim, const AttnPlan& pl, hipStream_t stream);
}  // namespace tva

namespace {

#ifndef JK_SPREAD
#define JK_SPREAD 1
#endif
constexpr int kSpread = JK_SPREAD;  // score phases of a pipelined tile pair that carry the next round's transfers (0: none)

// The transfers of a round of full prefix tiles of a contiguous cache, one at a time: piece
// k = chunk k % N of tile k / N of the round.  Issued between the MFMAs of the tile loop: all
// waves of a workgroup leave the barrier together, and a burst of transfers from every wave
// queues up in front of the CU's one address unit (1 KB = 16 cycles each) while the waves
// wait to get rid of them with nothing else issued.
template <int D, int NW, int TPR>
struct RoundPieces {
  static constexpr int N = LaneChunks<D, NW>::N;
  static constexpr int PIECES = TPR * N;
  const uint16_t* base;  // first tile of the round
  long long tile_elems;
  unsigned slot;
  const LaneChunks<D, NW>* lc;
  __device__ __forceinline__ void issue(int k) const {
    const int w = k / N, i = k % N;
    dma16(base + w * tile_elems, lc->off[i], slot + w * 2 * Geo<D>::TILE_BYTES + lc->lds[i]);
  }
  // pieces [P * step / steps, P * (step + 1) / steps): an even share for each of `steps` places
  __device__ __forceinline__ void share(int step, int steps) const {
    // (fenced: left alone, the compiler gathers the MFMAs in front of the transfers)
    if (PIECES * step / steps < PIECES * (step + 1) / steps) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < PIECES; ++k)
      if (k >= PIECES * step / steps && k < PIECES * (step + 1) / steps) issue(k);
    if (PIECES * step / steps < PIECES * (step + 1) / steps) __builtin_amdgcn_sched_barrier(0);
  }
};

// Per-wave state of the online softmax and the output accumulation (32 query rows).
template <int D>
struct WaveState {
  bf16x8 q[Geo<D>::DK];
  floatx16 o[Geo<D>::DB];
  float m, l;
};

// S^T = K . Q^T of KT consecutive 32-key tiles (K tiles 2*TILE_BYTES apart in LDS) against
// the wave's 32 query rows.  A chain of MFMAs into one accumulator issues only every other
// MFMA slot (each waits for its predecessor's result), so two independent chains are kept in
// flight: the two tiles' (KT = 2), or the even and odd k-steps of the one tile, summed at
// the end (KT = 1).
template <int D, int KT>
__device__ __forceinline__ void qk_tiles(const WaveState<D>& st, unsigned k_addr, floatx16& s0, floatx16& s1) {
  using G_ = Geo<D>;
  floatx16 a0, a1;
#pragma unroll
  for (int i = 0; i < 16; ++i) a0[i] = a1[i] = 0.f;
  if (KT == 2) {
#pragma unroll
    for (int ks = 0; ks < G_::DK; ++ks) {
      const bf16x8 k0 = lds_read128(k_addr ^ (ks << 5));
      const bf16x8 k1 = lds_read128((k_addr ^ (ks << 5)) + 2 * G_::TILE_BYTES);
      a0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k0, st.q[ks], a0, 0, 0, 0);
      a1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k1, st.q[ks], a1, 0, 0, 0);
    }
    s0 = a0;
    s1 = a1;
  } else {
#pragma unroll
    for (int ks = 0; ks < G_::DK; ks += 2) {
      const bf16x8 k0 = lds_read128(k_addr ^ (ks << 5));
      const bf16x8 k1 = lds_read128(k_addr ^ ((ks + 1) << 5));
      a0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k0, st.q[ks], a0, 0, 0, 0);
      a1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k1, st.q[ks + 1], a1, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) s0[i] = a0[i] + a1[i];
  }
}

// Online softmax and O^T += V^T . P^T for the KT tiles of a round whose (masked) scores are
// in s0 (and s1); v0 / v1 are their V tiles in LDS.  Two tiles share one running-maximum
// update, and their independent MFMA chains fill each other's latencies.
template <int D, int KT>
__device__ __forceinline__ void softmax_probs(WaveState<D>& st, const floatx16& s0, const floatx16& s1,
                                              float scale_log2, bf16x8 (&pb)[2 * KT]) {
  using G_ = Geo<D>;
  constexpr int DB = G_::DB;
  // The reference maximum m of a row moves only when the round's maximum exceeds it by more
  // than kLazy (in log2 units): weights then stay below 2^kLazy, harmless in fp32/bf16, and
  // the rescale of the accumulators becomes rare.  The result is unchanged: weights, their
  // sum and the accumulators all carry the same reference.
  constexpr float kLazy = 8.f;
  float tmax = max16(s0);
  if (KT == 2) tmax = fmaxf(tmax, max16(s1));
  tmax = half_swap_max(tmax) * scale_log2;
  const float m_old = st.m;
  const bool up = tmax > m_old + kLazy;  // false for tmax = -inf; true for the first visible key
  const float m_ref = up ? tmax : m_old;
  const float m_use = (m_ref == -INFINITY) ? 0.f : m_ref;
  const float alpha = up ? fast_exp2(m_old - m_use) : 1.f;
  const bool moved = up && (m_old != -INFINITY);  // accumulators are still zero before the first key
  st.m = m_ref;
  // probabilities become bf16 B operands of the value product
  float lsum = 0.f;
#pragma unroll
  for (int kt = 0; kt < KT; ++kt)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float sc = kt == 0 ? s0[8 * j + e] : s1[8 * j + e];
        const float pr = fast_exp2(fmaf(sc, scale_log2, -m_use));
        lsum += pr;
        pb[2 * kt + j][e] = (__bf16)pr;
      }
  st.l = fmaf(st.l, alpha, lsum);
  if (__any(moved)) {
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) st.o[db][i] *= alpha;
  }
}

template <int D, int KT>
__device__ __forceinline__ void softmax_pv(WaveState<D>& st, const floatx16& s0, const floatx16& s1,
                                           unsigned v_addr, float scale_log2) {
  using G_ = Geo<D>;
  constexpr int DB = G_::DB;
  bf16x8 pb[2 * KT];
  softmax_probs<D, KT>(st, s0, s1, scale_log2, pb);
  // ---- O^T += V^T . P^T
#pragma unroll
  for (int kt = 0; kt < KT; ++kt)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const bf16x8 vf = lds_read_tr2((v_addr ^ (db << 6)) + kt * 2 * G_::TILE_BYTES + 16 * j * G_::ROW_BYTES,
                                       8 * G_::ROW_BYTES);
        st.o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pb[2 * kt + j], st.o[db], 0, 0, 0);
      }
}

// Two unmasked tiles A, B of a round, software-pipelined by hand.  Within one tile the score
// product (MFMA), the softmax (vector ALU, a quarter-rate exponential per score) and the
// value product (MFMA) depend on each other, and a lone wave on its SIMD issues in order: it
// would use the two units one after the other.  Here the vector work of one tile is written
// between the MFMAs of the other:
//   S(A) | softmax(A) with S(B) | softmax(B) with O += P(A) V(A) | O += P(B) V(B)
template <int D>
struct PairPipe {
  using G_ = Geo<D>;
  static constexpr int DK = G_::DK, DB = G_::DB;
  // The pipelined pair never rescales the accumulators.  A row's reference m is fixed by the
  // first tile it sees (its maximum) or by the general path (which moves it, lazily, with a
  // rescale), and probabilities 2^(s - m) are allowed to grow: bf16 and fp32 have eight
  // exponent bits, so weights up to 2^kFrame lose no precision, and sums over 2^24 keys stay
  // far below 2^127.  A conditional rescale of the 64 accumulator registers inside the pair
  // costs the path that skips it a copy of all of them per tile pair (the compiler gives the
  // rescaled block new registers) and 64 registers of pressure where it sits.  A score more
  // than 2^kFrame above the reference (about 44 nats: a degenerate softmax) raises `left`;
  // the workgroup then repeats its whole split on the general path (see the tile loop).
  static constexpr float kFrame = 64.f;
  // The reference of a row: the maximum of the first tile its split sees (FIRST: nothing has been
  // accumulated for any row of the wave yet), kept from then on.  Later tiles do not even look for
  // their maximum: a weight beyond 2^kFrame shows in the row's sum, which the tile loop tests once,
  // after the last tile (left_frame below).
  static __device__ __forceinline__ float reference(WaveState<D>& st, const floatx16& s, float scale_log2, bool first) {
    if (!first) return st.m;  // (uniform)
    const float tmax = half_swap_max(max16(s)) * scale_log2;  // (an unmasked tile of finite scores: finite)
    const float m = (st.m == -INFINITY) ? tmax : st.m;
    st.m = m;
    return m;
  }
  // whether a weight of this lane's row went beyond 2^kFrame (or was NaN): its sum tells
  static __device__ __forceinline__ bool left_frame(const WaveState<D>& st) { return !(st.l < 1.8446744e19f); }

  // two scores -> probabilities (elements 2*i, 2*i+1 of the tile) into their bf16 operand slot; the
  // row sum takes the rounded probabilities (one dot product with (1, 1) instead of two additions,
  // and numerator and denominator of the softmax then carry the same rounding)
  static __device__ __forceinline__ void two_probs(const floatx16& s, int i, float scale_log2, float m_use,
                                                   float& lsum, bf16x8 (&pb)[2]) {
    const float p0 = fast_exp2(fmaf(s[2 * i], scale_log2, -m_use));
    const float p1 = fast_exp2(fmaf(s[2 * i + 1], scale_log2, -m_use));
    bf16x2 pk, one;
    pk[0] = (__bf16)p0;
    pk[1] = (__bf16)p1;
    one[0] = one[1] = (__bf16)1.f;
    lsum = __builtin_amdgcn_fdot2_f32_bf16(pk, one, lsum, false);
    pb[(2 * i) / 8][(2 * i) % 8] = pk[0];
    pb[(2 * i) / 8][(2 * i) % 8 + 1] = pk[1];
  }

  // k_addr / v_addr: LDS byte address of tile A's K / V tile plus the lane's Geo::k_lane / v_lane
  // `next`: the transfers of the round that refills the ring (SPREAD > 0), issued between the
  // MFMAs of the first SPREAD score phases
  // `first`: the wave's first tiles of its split (uniform)
  template <int SPREAD, class Pieces>
  static __device__ __forceinline__ void run(WaveState<D>& st, unsigned k_addr, unsigned v_addr, float scale_log2,
                                             const Pieces& next, bool first) {
    static_assert(DK == 8 || DK == 4, "head_dim 128 or 64");
    constexpr unsigned kNextTile = 2 * G_::TILE_BYTES;  // tile B's K (V) tile follows tile A's K and V
    auto v_frag = [&](unsigned tile_off, int j, int db) {
      return lds_read_tr2((v_addr ^ (db << 6)) + tile_off + 16 * j * G_::ROW_BYTES, 8 * G_::ROW_BYTES);
    };
    // LDS operands are fetched a whole phase ahead of the MFMAs that use them: a read issued
    // just before its MFMA would expose the LDS latency eight times per phase
    bf16x8 kf[DK], vfA[2 * DB], vfB[2 * DB];

    // ---- S(A), and between its MFMAs the transfers of the next round
    floatx16 sA, sB;
#pragma unroll
    for (int i = 0; i < 16; ++i) sA[i] = sB[i] = 0.f;
#pragma unroll
    for (int ks = 0; ks < DK; ++ks) kf[ks] = lds_read128(k_addr ^ (ks << 5));
#pragma unroll
    for (int ks = 0; ks < DK; ++ks) {
      sA = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], st.q[ks], sA, 0, 0, 0);
      if (SPREAD > 0) next.share(ks, DK * SPREAD);
    }
    // (scheduling fences between the phases: left alone, the compiler hoists the next phase's
    // LDS reads above this phase and runs out of registers)
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < DK; ++ks) kf[ks] = lds_read128((k_addr ^ (ks << 5)) + kNextTile);  // lands while the chain drains

    // ---- softmax(A) between the MFMAs of S(B).  The first half of S(B) is issued ahead of
    // the running-maximum update of A (a chain of dependent vector instructions that waits
    // for the last MFMA of S(A)): the matrix unit works through them meanwhile.
    bf16x8 pA[2], pB[2];
    float lsum = 0.f;
#pragma unroll
    for (int ks = 0; ks < DK / 2; ++ks) {
      sB = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], st.q[ks], sB, 0, 0, 0);
      if (SPREAD > 1) next.share(DK + ks, DK * SPREAD);
    }
    __builtin_amdgcn_sched_barrier(0);
    const float mA = reference(st, sA, scale_log2, first);
#pragma unroll
    for (int ks = DK / 2; ks < DK; ++ks) {
      sB = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], st.q[ks], sB, 0, 0, 0);
      if (SPREAD > 1) next.share(DK + ks, DK * SPREAD);
#pragma unroll
      for (int i = (ks - DK / 2) * (16 / DK); i < (ks - DK / 2 + 1) * (16 / DK); ++i)
        two_probs(sA, i, scale_log2, mA, lsum, pA);
    }
    st.l += lsum;
    __builtin_amdgcn_sched_barrier(0);

    // ---- softmax(B) between the MFMAs of O += V(A)^T . P(A)^T, in the same way.  The V
    // fragments of B are requested with those of A and arrive under this phase.
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int db = 0; db < DB; ++db) vfA[j * DB + db] = v_frag(0, j, db);
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int db = 0; db < DB; ++db) vfB[j * DB + db] = v_frag(kNextTile, j, db);
#pragma unroll
    for (int db = 0; db < DB; ++db)
      st.o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vfA[db], pA[0], st.o[db], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    lsum = 0.f;
    const float mB = mA;  // (the reference is fixed by now)
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      st.o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vfA[DB + db], pA[1], st.o[db], 0, 0, 0);
#pragma unroll
      for (int i = db * (8 / DB); i < (db + 1) * (8 / DB); ++i) two_probs(sB, i, scale_log2, mB, lsum, pB);
    }
    st.l += lsum;
    __builtin_amdgcn_sched_barrier(0);

    // ---- O += V(B)^T . P(B)^T
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int db = 0; db < DB; ++db)
        st.o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vfB[j * DB + db], pB[j], st.o[db], 0, 0, 0);
  }
};

// One unmasked tile on its own: the odd last tile of a split of the 4x1 arrangement (everybody
// else waits for the splits that have one).  All LDS operands are requested before the first
// MFMA, the K fragments first: the V fragments then arrive under the score product and the
// softmax instead of in front of the value product.  Same fixed reference frame as the
// pipelined pair: no rescale of the accumulators here.  (For the one-tile rounds of the 2x2
// arrangement this path measured slower than the general one - 63 registers more, and those
// shapes are not bound by the tile arithmetic.)
template <int D>
__device__ __forceinline__ void lone_tile(WaveState<D>& st, unsigned k_addr, unsigned v_addr, float scale_log2,
                                          bool first) {
  using G_ = Geo<D>;
  constexpr int DK = G_::DK, DB = G_::DB;
  bf16x8 kf[DK], vf[2 * DB];
#pragma unroll
  for (int ks = 0; ks < DK; ++ks) kf[ks] = lds_read128(k_addr ^ (ks << 5));
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int db = 0; db < DB; ++db)
      vf[j * DB + db] = lds_read_tr2((v_addr ^ (db << 6)) + 16 * j * G_::ROW_BYTES, 8 * G_::ROW_BYTES);
  __builtin_amdgcn_sched_barrier(0);
  floatx16 a0, a1, s0;
#pragma unroll
  for (int i = 0; i < 16; ++i) a0[i] = a1[i] = 0.f;
#pragma unroll
  for (int ks = 0; ks < DK; ks += 2) {  // two chains: a dependent MFMA issues only every other slot
    a0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], st.q[ks], a0, 0, 0, 0);
    a1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks + 1], st.q[ks + 1], a1, 0, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) s0[i] = a0[i] + a1[i];
  const float m = PairPipe<D>::reference(st, s0, scale_log2, first);
  bf16x8 pb[2];
  float lsum = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) PairPipe<D>::two_probs(s0, i, scale_log2, m, lsum, pb);
  st.l += lsum;
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int db = 0; db < DB; ++db)
      st.o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[j * DB + db], pb[j], st.o[db], 0, 0, 0);
}

// Profiling build only (-DJK_TIMING, not part of the shipped library): thread 0 of every
// workgroup records the 100 MHz wall clock at points of the kernel (entry, speculative
// transfers issued, prefix length known, transfers issued, first round landed, loop done,
// columns parked, partials stored, arrived at the group word, group complete, end); jk_debug_read_timing<JK_MERGE> copies the table of the last launch to the host
// (grids of at most 4096 workgroups).  Phase times of the kernel are measured with it.
#ifdef JK_TIMING
__device__ unsigned long long g_jk_ts[4096 * 16];
#define JK_TS(i) do { if (threadIdx.x == 0) g_jk_ts[blockIdx.x * 16 + (i)] = wall_clock64(); } while (0)
#else
#define JK_TS(i) do { } while (0)
#endif

// ---------------------------------------------------------------- split merge inside the kernel
// The workgroups that hold the S key splits of one (unit, row tile) group all run on one XCD
// (the host only asks for this path when its workgroup numbering guarantees it and the
// device's round-robin placement has been verified), so they can meet in that XCD's L2
// without the whole-cache write-back an agent-scope release costs on a part with eight L2s:
// partials are written with ordinary stores (a CU's vector cache writes through to L2; a
// store is acknowledged, and counted off vmcnt, once L2 has it), arrivals are counted with
// atomics that carry no device scope and therefore execute in that L2, and the partials are
// read back with loads that miss the reader's vector cache (invalidated first).  This is the
// hardware's own recipe for workgroup-scope synchronisation between CUs that share an L2.
__device__ __forceinline__ unsigned l2_atomic_add(unsigned* p, unsigned x) {
  unsigned v;
  asm volatile("global_atomic_add %0, %1, %2, off sc0\n\ts_waitcnt vmcnt(0)" : "=v"(v) : "v"(p), "v"(x) : "memory");
  return v;
}
__device__ __forceinline__ unsigned l2_atomic_or(unsigned* p, unsigned x) {
  unsigned v;
  asm volatile("global_atomic_or %0, %1, %2, off sc0\n\ts_waitcnt vmcnt(0)" : "=v"(v) : "v"(p), "v"(x) : "memory");
  return v;
}
__device__ __forceinline__ unsigned l2_atomic_swap(unsigned* p, unsigned x) {
  unsigned v;
  asm volatile("global_atomic_swap %0, %1, %2, off sc0\n\ts_waitcnt vmcnt(0)" : "=v"(v) : "v"(p), "v"(x) : "memory");
  return v;
}
__device__ __forceinline__ void l2_atomic_add_noret(unsigned* p, unsigned x) {
  asm volatile("global_atomic_add %0, %1, off" ::"v"(p), "v"(x) : "memory");
}

// Merge of rows [slice * R, (slice + 1) * R) of the group's row tile over all S splits, written to
// the output.  16 bytes (8 columns) of a row per thread; the arithmetic per element is that of the
// stand-alone merge kernel (splits in chunks of 8, running maximum), so both give the same bits.
struct MergeArgs {
  const float* part_o;
  const float2* part_ml;
  uint16_t* out;
  int M, m_pad, splits, G;
  unsigned long long mg_g;
  long long o_sb, o_st, o_sh;
};
// Reductions over aligned groups of 2^sh lanes (sh uniform): within a row of 16 lanes by DPP
// (quad permutes, then the mirrors of 8 and of 16 lanes: after the quads every lane of a quad
// holds the quad's value, so a mirror pairs quads as well as an exchange would), across rows by shuffles.
template <int CTRL>
__device__ __forceinline__ float dpp_f(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float group_max(float x, int sh) {
  if (sh >= 1) x = fmaxf(x, dpp_f<0xB1>(x));   // quad_perm [1,0,3,2]
  if (sh >= 2) x = fmaxf(x, dpp_f<0x4E>(x));   // quad_perm [2,3,0,1]
  if (sh >= 3) x = fmaxf(x, dpp_f<0x141>(x));  // row_half_mirror
  if (sh >= 4) x = fmaxf(x, dpp_f<0x140>(x));  // row_mirror
  if (sh >= 5) x = fmaxf(x, __shfl_xor(x, 16));
  if (sh >= 6) x = fmaxf(x, __shfl_xor(x, 32));
  return x;
}
__device__ __forceinline__ float group_sum(float x, int sh) {
  if (sh >= 1) x += dpp_f<0xB1>(x);
  if (sh >= 2) x += dpp_f<0x4E>(x);
  if (sh >= 3) x += dpp_f<0x141>(x);
  if (sh >= 4) x += dpp_f<0x140>(x);
  if (sh >= 5) x += __shfl_xor(x, 16);
  if (sh >= 6) x += __shfl_xor(x, 32);
  return x;
}

// Merge of one slice (R consecutive rows of a row tile) over all S splits, written to the output:
//   m = max_s m_s,  l = sum_s l_s 2^(m_s - m),  out = sum_s O_s 2^(m_s - m) / l.
// What limits it is the issue rate of a lone wave per SIMD (about eight cycles an instruction)
// and the CU's one path to L2, so: everything that does not depend on the partials (row numbers,
// byte offsets, the output address) is worked out by merge_prepare while the workgroup still
// waits for its partners; then (A) one thread per (row, split) fetches that pair's (max, sum)
// once, the 2^sh lanes of a row find the row's maximum and sum and park the normalised weight
// 2^(m_s - m) / l in LDS, while (B) one thread per (row, 4 columns) has its 8 (fp32: 16) bytes of every
// split's partial in flight and afterwards only multiplies and adds.  At most THREADS (row, split)
// pairs exist per slice (R = ceil(tile rows / S), S padded to 2^sh), one per thread.  FINE: the partials are fp32.
struct MergeThread {
  unsigned raw_off;   // byte offset of this thread's 4 columns in split 0's partial (rows of the first pass)
  unsigned ml_off;    // byte offset of this thread's (row, split) pair
  unsigned dst_off;   // element offset of this thread's 4 output columns in `out` (first pass)
  unsigned unit_end;  // rows of partials up to the end of the unit's
  int r_b, row_lo, row_hi;
  bool live_a;
};

template <int D, int THREADS, int QROWS, bool FINE>
__device__ __forceinline__ MergeThread merge_prepare(const MergeArgs& p, int unit_id, int b, int kv, int slice, int R,
                                                     int sh, int tile_row0, int tid) {
  constexpr int CPR = D / 4;
  MergeThread t;
  const int S = p.splits;
  t.row_lo = slice * R;
  t.row_hi = min(QROWS, t.row_lo + R);
  const int chunk = tid % CPR;
  t.r_b = t.row_lo + tid / CPR;
  const unsigned unit_row0 = (unsigned)(unit_id * S) * (unsigned)p.m_pad + (unsigned)tile_row0;  // (the host keeps
  t.unit_end = (unsigned)((unit_id + 1) * S) * (unsigned)p.m_pad;                                // the partials below 2^31 bytes)
  t.raw_off = ((unit_row0 + (unsigned)t.r_b) * (unsigned)D + (unsigned)chunk * 4u) * (FINE ? 4u : 2u);
  const int ra = t.row_lo + (tid >> sh), sa = tid & ((1 << sh) - 1);
  t.live_a = ra < t.row_hi && tile_row0 + ra < p.M && sa < S;
  // (a lane without a pair asks for one of its own group's: a line of another group's, read before that one is complete, would
  // stay in this CU's vector cache for the workgroup that merges it)
  t.ml_off = (t.live_a ? unit_row0 + (unsigned)ra + (unsigned)sa * (unsigned)p.m_pad : unit_row0) * 8u;
  const int m = min(tile_row0 + t.r_b, p.M - 1);
  const int node = div_mg(m, p.mg_g);
  t.dst_off = (unsigned)(b * p.o_sb + node * p.o_st + (long long)(kv * p.G + (m - node * p.G)) * p.o_sh) + chunk * 4;
  return t;
}

// (B) for up to 2^SH splits at a time, of as many rows as a thread's sixteen slots hold: all of a slice's rows
// go out together (a 128-row tile in 2^k splits leaves a thread exactly 16 / 2^k of them).  One row after the other,
// each a round trip to L2, two splits of a 4x1 workgroup took 5.7 us longer to merge than sixteen.
template <int D, int THREADS, int QROWS, int SH, bool FINE>
__device__ __forceinline__ void merge_rows(const MergeArgs& p, const MergeThread& t, int sh, int b, int kv, int tile_row0,
                                           int tid, float* wbuf) {
  constexpr int CPR = D / 4, RPP = THREADS / CPR, SP = SH < 4 ? 1 << SH : 16, ROWS = 16 / SP;
  const int S = p.splits;
  typedef std::conditional_t<FINE, u32x4, u32x2> Raw;
  constexpr unsigned ROW_BYTES = D * (FINE ? 4 : 2);
  const unsigned po_step = (unsigned)p.m_pad * ROW_BYTES;  // from one split's partial to the next
  const int rows_end = min(t.row_hi, p.M - tile_row0);
  // (The unit's partials end where the buffer does: what a padded split or a row past the slice would read is zeros, without a
  // condition.  With a branch for each of the sixteen loads, and the code in front of them that the compiler made of those,
  // a layer of an 8B model, 4096 keys in sixteen splits, had its rows' weights 1.7 us after the group was complete, and has
  // them after 0.9 like this; the step of 32 such layers takes 456 us instead of 469.)
  const auto part = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.part_o), 0, t.unit_end * ROW_BYTES, 0x00020000);
  constexpr unsigned kNowhere = 0x80000000u;  // (merged here are at most two workgroups a CU: tens of megabytes)
  Raw raw[16];
  auto fetch = [&](int r0, int s0) {
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
      const int r = r0 + k * RPP;
      unsigned off = r < rows_end ? t.raw_off + (unsigned)s0 * po_step + (unsigned)(r - t.r_b) * ROW_BYTES : kNowhere;
      asm volatile("" : "+v"(off));  // (one addition a load: left alone, the compiler makes sixteen induction variables of the loop
                                     // over left slices, ninety instructions in front of it)
#pragma unroll
      for (int u = 0; u < SP; ++u) {
        if constexpr (FINE) raw[k * SP + u] = __builtin_amdgcn_raw_buffer_load_b128(part, (int)off, 0, 0);
        else raw[k * SP + u] = __builtin_amdgcn_raw_buffer_load_b64(part, (int)off, 0, 0);
        off += po_step;
      }
    }
  };
  // ---- the (max, sum) pair of this thread's (row, split) first, then (B), first half
  // (The pair is loaded by hand and waited for by number, with the sixteen loads behind it on their way: left alone, the
  // compiler waits in front of them, or for all of them.)
  u32x2 pair;
  asm volatile("global_load_dwordx2 %0, %1, %2 ; asked %0 as %3" : "=v"(pair) : "v"(t.ml_off), "s"(p.part_ml), "n"(kAskedPair) : "memory");
  const bool rows_here = __builtin_amdgcn_readfirstlane(t.r_b) < rows_end;  // (of this wave: its first row is its least)
  if (rows_here) {
    fetch(t.r_b, 0);
    dev::wait_vm<16>();
  } else {
    dev::wait_vm<0>();
  }
  arrived<kAskedPair>(pair);
  const float2 ml = t.live_a ? make_float2(__uint_as_float(pair[0]), __uint_as_float(pair[1])) : make_float2(-INFINITY, 0.f);
  JK_TS(11);
  // ---- (A): pair (row, split) of this thread
  const int wsh = sh < 2 ? 2 : sh;  // (a row's weights start at a multiple of four floats, for the 16-byte reads below)
  {
    const float top = dev::part_top(ml.x, ml.y);
    const float mx = group_max(top, sh);
    const float w = fast_exp2(top - ((mx == -INFINITY) ? 0.f : mx));  // exp2(-inf) = 0
    const float l = group_sum(ml.y * w, sh);
    // (l > 0 for a live row: it sees at least its own tree key; dead rows are not stored)
    wbuf[((tid >> sh) << wsh) | (tid & ((1 << sh) - 1))] = w / l;
  }
  JK_TS(12);
  __syncthreads();
#ifdef JK_TIMING
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  JK_TS(13);
#endif
  // ---- (B), second half
  if (!rows_here) return;
  for (int r0 = t.r_b; r0 < t.row_hi; r0 += ROWS * RPP) {
    float acc[ROWS][4];
#pragma unroll
    for (int k = 0; k < ROWS; ++k) acc[k][0] = acc[k][1] = acc[k][2] = acc[k][3] = 0.f;
    for (int s0 = 0; s0 < (SH < 5 ? 1 : S); s0 += SP) {  // (SH < 5: no more than SP splits)
      if (r0 != t.r_b || s0 > 0) fetch(r0, s0);  // (beyond what went out above)
#pragma unroll
      for (int k = 0; k < ROWS; ++k) {
        // (a row past the slice reads another row's weights or none: its data are zeros and it is not stored)
        const float* wrow = wbuf + ((min(r0 + k * RPP, t.row_hi - 1) - t.row_lo) << wsh) + s0;
#pragma unroll
        for (int u = 0; u < SP; u += 4) {
          const float4 w4 = *reinterpret_cast<const float4*>(wrow + u);
          const float w[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
          for (int v = 0; v < 4 && u + v < SP; ++v) {
            const Raw x = raw[k * SP + u + v];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              unsigned bits;
              if constexpr (FINE) bits = x[e];
              else bits = (e & 1) ? x[e / 2] & 0xffff0000u : x[e / 2] << 16;
              acc[k][e] = fmaf(__uint_as_float(bits), w[v], acc[k][e]);
            }
          }
        }
      }
    }
#pragma unroll
    for (int k = 0; k < ROWS; ++k) {
      const int r = r0 + k * RPP;
      if (r >= rows_end) continue;
      u32x2 pk;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        bf16x2 o;
        o[0] = (__bf16)acc[k][2 * h];
        o[1] = (__bf16)acc[k][2 * h + 1];
        pk[h] = __builtin_bit_cast(unsigned, o);
      }
      uint16_t* dst;
      if (k == 0 && r0 == t.r_b) {
        dst = p.out + t.dst_off;
      } else {
        const int m = tile_row0 + r;
        const int node = div_mg(m, p.mg_g);
        dst = p.out + b * p.o_sb + node * p.o_st + (long long)(kv * p.G + (m - node * p.G)) * p.o_sh + (tid % CPR) * 4;
      }
      *reinterpret_cast<u32x2*>(dst) = pk;  // (an ordinary store measured no slower than one through to memory here)
    }
  }
}

// The kernel's arguments in front of its KParams: what a wave needs first, fourteen words, as many as the hardware puts into scalar registers
struct LeadingArgs {
  const int32_t* prefix_len;
  int batch, total_wgs, n_qtiles, splits, units_per_xcd, second_turn, n_kv_heads;
  unsigned mg_qtiles, mg_splits, mg_hkv, mg_upx;  // the lower halves of KParams'
};
constexpr int kParamsAt = (sizeof(LeadingArgs) + 7) / 8 * 8;
// n / d, mg the lower half of what div_mg takes
__device__ __forceinline__ int divide(int n, unsigned mg, int d) { return d == 1 ? n : (int)__umulhi((unsigned)n, mg); }

// LDS plan of one workgroup, shared by the kernel and its launcher.
template <int D, int WM, int WN, int KT, bool PAGED = false, bool DEEP = false>
struct Plan {
  using G_ = Geo<D>;
  static constexpr int NW = WM * WN;                    // waves
  static constexpr int THREADS = 64 * NW;
  static constexpr int TPR = WN * KT;                   // tiles per round: KT consecutive ones per key column
  // (deeper rings measured slower: with six tiles c3 +0.9 us per call, with eight +4.6 - more transfers in
  // flight at once delay the first round's data by more than the later rounds gain)
  // DEEP (2x2 only): six tiles, two rounds in flight.  For a lone workgroup per CU that does nothing but stream a
  // long prefix (few query rows, no splits: c6) 64 KB in flight instead of 32 measured 59.3 -> 56.1 us; where two
  // workgroups share a CU they have that much in flight between them, and the deeper ring, which lets only one
  // fit, measured slower (c7 23.3 -> 30.6 us, c2 12.1 -> 12.4)
  static constexpr int RING_TILES = TPR >= 4 ? 2 * TPR : (DEEP ? 6 : 4);  // K+V tile pairs resident in LDS
  static constexpr int NR = RING_TILES / TPR;           // rounds resident in the ring
  static constexpr int QROWS = kWaveRows * WM;
  static constexpr int STAGE_BYTES = TPR * 2 * G_::TILE_BYTES;  // one round: TPR tiles of K and V
  static constexpr int RING_BYTES = NR * STAGE_BYTES;
  static_assert(WN == 1 || WN == 2, "one key column, or two that share the epilogue");
  static constexpr int OB = G_::DB / WN, OCOLS = D / WN;  // 32-wide blocks (columns) of its rows that a wave finishes
  static constexpr int PARK_BYTES = 64 * OB * 64;  // two key columns: what one parks for a wave of the other
  static constexpr int PATCH_LD = OCOLS * 2 + 16;  // padded row of a wave's store patch: bf16, or half of the columns in fp32
  static constexpr int PATCH_BYTES = kWaveRows * PATCH_LD;
  static constexpr int SLOT_BYTES = WN == 2 ? PARK_BYTES : PATCH_BYTES;  // a wave's share of the epilogue's LDS
  static_assert(PATCH_BYTES <= SLOT_BYTES && NW * SLOT_BYTES <= (WN == 2 ? STAGE_BYTES : RING_BYTES), "the epilogue fits a slot of the ring (one key column: the ring)");
  static constexpr int ML_BYTES = NW * kWaveRows * 8;
  static constexpr int PAGES_BYTES = PAGED ? kMaxPagesPerSplit * 4 : 0;
  static constexpr int SMEM = RING_BYTES + ML_BYTES + JK_MAX_TREE * 16 + JK_MAX_TREE * 4 + 16 + PAGES_BYTES;
  static constexpr int WGS_PER_CU = 2 * SMEM <= 160 * 1024 && NW <= 4 ? 2 : 1;
  static constexpr int REG_WGS = NW <= 4 ? 2 : 1;  // register budget: at most 256 VGPRs, no detour through AGPRs
  static_assert(SMEM <= 160 * 1024, "LDS budget");
  static_assert(THREADS >= JK_MAX_TREE, "one thread per tree node in the prologue");
};

// MERGE: see merge_of.  The host picks the instance, so that a kernel holds the code of one merge: with all four behind a switch (3400 instructions, and
// 113 - 146 scalar registers spilled, some of them in front of the tile loop) a layer of an 8B model, 4096 keys in sixteen
// splits, took 15.2 us, and 14.7 like this.
template <int D, int WM, int WN, int KT, bool PAGED, bool DEEP, int MERGE>
__global__ __launch_bounds__((Plan<D, WM, WN, KT, PAGED, DEEP>::THREADS), (Plan<D, WM, WN, KT, PAGED, DEEP>::REG_WGS)) void tva_bf16_kernel(
    const int32_t* prefix_len, int batch, int total_wgs, int n_qtiles, int splits, int units_per_xcd, int second_turn, int n_kv_heads,
    unsigned mg_qtiles, unsigned mg_splits, unsigned mg_hkv, unsigned mg_upx, const KParams p) {
  using G_ = Geo<D>;
  using P_ = Plan<D, WM, WN, KT, PAGED, DEEP>;
  constexpr int TPR = P_::TPR;
  constexpr int DK = G_::DK, DB = G_::DB;
  constexpr int NW = P_::NW, THREADS = P_::THREADS, NR = P_::NR, QROWS = P_::QROWS;
  constexpr int TILE_BYTES = G_::TILE_BYTES;
  constexpr int STAGE_BYTES = P_::STAGE_BYTES;
  constexpr int DMA_PER_ROUND = TPR * LaneChunks<D, NW>::N;  // transfers a wave issues per round
  static_assert(NR >= 2 && (NR - 2) * DMA_PER_ROUND <= 63, "wave arrangement");

  constexpr bool FINE = MERGE == 1 || MERGE == 2;  // partials merged here are fp32

  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];  // the kernel has no other LDS: offset 0
  unsigned char* ring = smem;
  float2* mlbuf = reinterpret_cast<float2*>(smem + P_::RING_BYTES);              // [NW][32]
  unsigned long long* anc = reinterpret_cast<unsigned long long*>(smem + P_::RING_BYTES + P_::ML_BYTES);  // [128][2]
  int* par_s = reinterpret_cast<int*>(smem + P_::RING_BYTES + P_::ML_BYTES + JK_MAX_TREE * 16);           // [128]
  int* repeat_s = par_s + JK_MAX_TREE;  // set by a wave whose scores left the pipelined pairs' fixed reference frame
  int* pg_s = repeat_s + 4;             // [1024], paged caches only

  JK_TS(0);
  // ---- The leading arguments are in scalar registers when a wave starts (a compiler option for this file): which piece of work
  // this is, and the lengths' address.  The others take 0.25 us to come from memory, for which their 64-byte lines are
  // touched at once: the compiler fetches them in several dependent batches, and this way only the first pays the trip.
  typedef __attribute__((address_space(4))) const unsigned kernarg_word;
  kernarg_word* ka = (kernarg_word*)__builtin_amdgcn_kernarg_segment_ptr();
  static_assert(kParamsAt == 56 && sizeof(LeadingArgs) <= 56 && sizeof(KParams) > 328 && sizeof(KParams) <= 392, "seven lines of kernel arguments");
  const unsigned a0 = ka[14], a1 = ka[16], a2 = ka[32], a3 = ka[48], a4 = ka[64], a5 = ka[80], a6 = ka[96];
  __builtin_amdgcn_sched_barrier(0);
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % WM;
  const int wn = wave / WM;
  const int c32 = lane & 31;
  const int g = lane >> 5;
  // (what needs no argument is worked out while they are on their way)
  unsigned column = lane_column<D, NW>(wave, lane);
  // (A wave of key column 1 takes the blocks of the head dimension second half first: its first accumulators then are the
  // half that it finishes, and no register is chosen by the wave.)
  unsigned k_lane = G_::k_lane(lane), v_lane = G_::v_lane(lane) ^ ((unsigned)(wn * P_::OB) << 6);
  asm volatile("" : "+v"(column), "+v"(k_lane), "+v"(v_lane));
  // ---- which piece of work: consecutive hardware workgroup ids alternate between the 8
  // XCDs, so give each XCD a contiguous range of logical ids; q-tiles of one (b, kv, split)
  // are adjacent logical ids and therefore share that XCD's L2 for their common K/V.
  // In a batch the (sequence, KV head) units are put in order of falling length, which only the device knows, and dealt
  // to the XCDs in turn (every other time backwards): each XCD gets its share of long and short sequences, starts with
  // the long ones, and where the grid is two workgroups a CU the second 32 of an XCD come the other way round, so that
  // the longest shares its CU with the shortest.  16 sequences of 512 to 4096 tokens (8B shapes) took 88 us in the
  // order of the batch (an XCD had two sequences of its own), 67 like this.
  const bool ranked = units_per_xcd > 0;
  // The prefix length first.  Ordinary loads are issued by hand like the transfers behind them, and waited for by number: the
  // compiler, which does not know of the transfers, would wait for the oldest of its loads by waiting for all but a few of
  // everything issued since.
  int lengths;  // (lane i: of sequence i, of the first 64)
  load_by_hand<kAskedLengths>(lengths, prefix_len + min(lane, batch - 1));
  int wid;
  {
    const int n = blockIdx.x;
    const int per = total_wgs >> 3;  // total_wgs is padded to a multiple of 8
    int local = n >> 3;
    if (ranked && local >= second_turn) local = second_turn + per - 1 - local;
    wid = (n & 7) * per + local;
  }
  const int rest = divide(wid, mg_qtiles, n_qtiles);
  const int qtile = wid - rest * n_qtiles;
  const int unit = divide(rest, mg_splits, splits);  // b * Hkv + kv in the order of the batch
  if (unit >= batch * n_kv_heads) return;    // padding workgroup (a wave's end waits for what it has asked for)
  const int split = rest - unit * splits;
  int place = unit;  // rank * Hkv + kv
  if (ranked) {
    const int x = divide(unit, mg_upx, units_per_xcd), i = unit - x * units_per_xcd;
    place = i * 8 + ((i & 1) ? 7 - x : x);
  }
  const int rank = divide(place, mg_hkv, n_kv_heads);
  const int kv = place - rank * n_kv_heads;
  int b = rank;  // (a ranked batch: until the lengths are there)
  // ---- from here on with the arguments that had to come
  {
    int r = rank, q = qtile, s = split;
    asm volatile("" : "+s"(r), "+s"(q), "+s"(s));
    asm volatile("" ::"s"(a0), "s"(a1), "s"(a2), "s"(a3), "s"(a4), "s"(a5), "s"(a6));
  }
  const int T = p.T, G = p.G, M = p.M;
  const float scale_log2 = p.scale_log2;
  const int m_row = qtile * QROWS + wm * kWaveRows + c32;  // this lane's query row
  const bool row_ok = m_row < M;
  const int mm = row_ok ? m_row : M - 1;  // (clamped: in bounds)
  const int my_node = div_mg(mm, p.mg_g);
  unsigned long long row_at = (unsigned)my_node * (unsigned long long)p.q_st + (unsigned)(kv * G + (mm - my_node * G)) * (unsigned long long)p.q_sh + 8 * g;
  int L = p.max_prefix, L_one;
  if (ranked) {
    asm volatile("" : "+v"(row_at));
    dev::wait_vm<0>();
    int len = taken<kAskedLengths>(lengths);
    len = len < 0 ? 0 : (len > p.max_prefix ? p.max_prefix : len);
    if (!__all(len == p.max_prefix)) {
      b = sequence_of_rank(len, batch, rank, lane);
      L = __builtin_amdgcn_readlane(len, b);
    }
  } else if (batch > 64) {
    load_by_hand<kAskedLength>(L_one, prefix_len + b);
  }
  JK_TS(14);

  // ---- tile range of this split.  A batch that is not ranked (one sequence, more than 64, or units that the XCDs cannot share out evenly): the
  // prefix length is still on its way, and the K/V stream starts on the assumption that it equals the host's upper bound; if it
  // turns out shorter, the speculative transfers are waited for and everything is redone.
  TileSrc ts;
  ts.T = T;
  ts.kc_sl = p.kc_sl;
  ts.kt_st = p.kt_st;
  ts.pg_s = pg_s;
  ts.pg_first = 0;
  ts.tpp = p.tpp;
  ts.mg_tpp = p.mg_tpp;
  ts.page_stride = p.page_stride;
  const int n_ttiles = (T + kTileKeys - 1) / kTileKeys;
  // Splits are dealt whole rounds (TPR tiles).  The rounds at the end of the key range that
  // hold the ragged prefix tile or masked tree tiles are slower (per-lane clamped transfers,
  // mask arithmetic, ancestor sets first), so each of them counts double when the rounds are
  // shared out (up to half of a split's share), the surplus going to the first splits: the
  // split that ends the range then finishes with the others instead of after them.
  auto set_range = [&](int len) {
    ts.L = len;
    ts.n_ptiles = (len + kTileKeys - 1) / kTileKeys;
    const int nt = ts.n_ptiles + n_ttiles;
    const int R = (nt + TPR - 1) / TPR;
    const int slow = R - (len / kTileKeys) / TPR;  // rounds that are not all full prefix tiles
    const int share = divide(R, mg_splits, splits);
    const int extra = slow < share / 2 ? slow : share / 2;
    const int Rv = R + extra;
    const int base = divide(Rv, mg_splits, splits);
    const int rem = Rv - base * splits;
    int rb = split * base + (split < rem ? split : rem);
    int re = rb + base + (split < rem ? 1 : 0);
    rb = rb < R ? rb : R;
    re = re < R ? re : R;
    ts.t_begin = rb * TPR < nt ? rb * TPR : nt;
    ts.t_end = re * TPR < nt ? re * TPR : nt;
    if (KT == 2 && WN == 1) {
      // One wave column taking tile pairs.  Everybody waits for the slowest split (the merge needs all
      // partials), so the shares are dealt in tiles of what the loop is fast at: full prefix tiles,
      // evenly (a split with an odd number ends on a lone tile, which costs about half a pair).  What
      // is left - the ragged tile, the masked tree tiles, all of them on the slower general path - goes
      // to the last split, priced at two full tiles a tile (measured: two tree tiles 2.8 us, a pair of
      // full tiles 1.31), and that split gets correspondingly fewer full tiles (none at all if the tail
      // is worth a whole share: the host may add a split for it, whose workgroups are short and share
      // a CU with a regular one).
      const int F = len / kTileKeys;  // full prefix tiles
      const int tail = nt - F;
      int tb = 0, te = nt;
      if (splits > 1) {
        const int per = divide(F + 2 * tail + splits - 1, mg_splits, splits);  // ceil((F + 2 tail) / splits)
        int f_last = per - 2 * tail;
        f_last = f_last < 0 ? 0 : (f_last > F ? F : f_last);
        f_last &= ~1;  // (whole pairs: the general path takes the tail two tiles at a time, and a full tile must not split one of its rounds)
        const int rest = F - f_last;  // full tiles of the other splits
        const int base_t = div_mg(rest, p.mg_splits_m1), rem_t = rest - base_t * (splits - 1);
        if (split == splits - 1) {
          tb = rest;
        } else {
          tb = split * base_t + (split < rem_t ? split : rem_t);
          te = tb + base_t + (split < rem_t ? 1 : 0);
        }
      }
      ts.t_begin = tb;
      ts.t_end = te;
    }
  };
  const unsigned ring_addr = (unsigned)(size_t)LDS_PTR(unsigned char, ring);  // a multiple of 1024
  LaneChunks<D, NW> lc;
  lane_chunks<D, NW>(lc, wave, lane, column, ts);
  const bool is_v = wave * LaneChunks<D, NW>::N >= G_::NB;
  lc.cache = uniform_ptr((is_v ? p.vc : p.kc) + (PAGED ? 0 : (unsigned)b * (unsigned long long)p.kc_sb) + (unsigned)kv * (unsigned long long)p.kc_sh);

  set_range(L);
  int n_rounds = (ts.t_end - ts.t_begin + TPR - 1) / TPR;
  // Paged cache: page ids of the prefix tiles this split will fetch (whole rounds), clamped into the pool, so
  // that a transfer stays inside the pool whatever the table holds: the first rounds can then be asked for on
  // the same assumption as with a contiguous cache (entries past a sequence's pages may hold anything; if the
  // length turns out shorter, the list is made again).  An id outside the pool is reported once the list is final.
  bool bad_page = false;
  int n_pg = 0, first_id;  // pages of the list; this thread's first entry
  const int* table = p.block_table + (long long)b * p.max_blocks;
  auto ask_pages = [&]() {
    const int te = min(ts.n_ptiles, ts.t_begin + n_rounds * TPR);
    n_pg = 0;
    if (te > ts.t_begin) {
      ts.pg_first = div_mg(ts.t_begin, p.mg_tpp);
      n_pg = div_mg(te - 1, p.mg_tpp) - ts.pg_first + 1;  // <= kMaxPagesPerSplit by the host's plan
    }
    // (in every lane: the compiler may not move the result before it has been waited for)
    load_by_hand<kAskedPages>(first_id, tid < n_pg && ts.pg_first + tid < p.max_blocks ? table + ts.pg_first + tid : p.prefix_len);
  };
  auto fill_pages = [&]() {  // (the ids have been waited for)
    arrived<kAskedPages>(first_id);
    bad_page = false;
    for (int i = tid; i < n_pg && i < kMaxPagesPerSplit; i += THREADS) {
      const int pi = ts.pg_first + i;
      const int id = pi >= p.max_blocks ? 0 : (i == tid ? first_id : table[pi]);
      bad_page = bad_page || id < 0 || id >= p.n_pages;
      pg_s[i] = id < 0 ? 0 : (id >= p.n_pages ? p.n_pages - 1 : id);
    }
    __syncthreads();
  };
  if (PAGED) ask_pages();  // (the query rows come while the page ids do)

  // ---- the query rows, and in the first wave, which builds the ancestor sets, the parents of nodes lane and lane + 64
  WaveState<D> st;
  u32x4 q_raw[DK];
  int parent_lo, parent_hi;
  {
    load_rows_by_hand<kAskedRow>(q_raw, p.q + (unsigned)b * (unsigned long long)p.q_sb + row_at);
    if (wave == 0) {
      const int32_t* parents = p.parent + (unsigned)(b * T);
      load_by_hand<kAskedParent>(parent_lo, parents + min(lane, T - 1));
      load_by_hand<kAskedParent + 1>(parent_hi, parents + min(lane + 64, T - 1));
    }
  }
  if (PAGED) {
    dev::wait_vm<DK>();
    fill_pages();
  }
  // ---- the first rounds.  (A ranked batch has its lengths by now.  Asked for as if all of them equalled the bound, which is seldom
  // so, the first rounds had to land before the right ones took their places.  us, so / like this: 8 sequences of up to 2048
  // keys, five nodes (8B shapes) 17.2 / 16.1, 12 of up to 900, 24 nodes 19.7 / 17.4, 4 of up to 2000, 60 nodes 22.2 / 20.8.  Lengths that do all
  // equal the bound can lose: in a grid of several turns the lengths come through a busy CU's memory queue, and the later workgroups have their
  // first tiles 4.7 us after their start, 4.1 before; in one turn the first tiles come earlier, 4.6 instead of 4.9, but all at once, and c4's loop, bound
  // by HBM, takes 26.3 instead of 25.7.  Whole calls with the shorter start and merge that came with it, lengths equal, and in brackets
  // ragged: 13 of 2519 keys, 12 nodes, 40 KV heads 137.5 / 139.5 (97.5 / 93.5), 16 of 123, 115 nodes, 40 KV heads 33.7 / 34.3 (33.8 / 31.6), 4 of
  // 2048, 60 nodes, 40 KV heads 42.5 / 42.9 (43.0 / 41.7), 5 of 1296, 43 nodes, heads of 64 10.9 / 11.0 (11.0 / 10.4); forty equal batches
  // together 1.016 times as fast, 0.981 to 1.08.)
  int n_spec = 0;  // rounds already issued, all of them full prefix tiles under the assumption
#pragma unroll
  for (int r = 0; r < NR - 1; ++r)
    if (n_spec == r && r < n_rounds && (ts.t_begin + (r + 1) * TPR) * kTileKeys <= L) {
      dma_round<D, NW, TPR, PAGED>(r, ts, lc, ring_addr + r * STAGE_BYTES);
      n_spec = r + 1;
    }
  JK_TS(1);
  // (not in front of the transfers, which are full prefix tiles)
  int b_late = b;
  asm volatile("" : "+s"(b_late));
  lc.tree = uniform_ptr((is_v ? p.vt : p.kt) + (unsigned)b_late * (unsigned long long)p.kt_sb + (unsigned)kv * (unsigned long long)p.kt_sh);
  if (!ranked) {
    if (n_spec == NR - 1) dev::wait_vm<DK + (NR - 1) * DMA_PER_ROUND>();
    else dev::wait_vm<DK>();  // (no less than needed)
    if (batch <= 64) L = __builtin_amdgcn_readlane(taken<kAskedLengths>(lengths), b);
    else L = __builtin_amdgcn_readfirstlane(taken<kAskedLength>(L_one));
    L = L < 0 ? 0 : (L > p.max_prefix ? p.max_prefix : L);
    JK_TS(2);
    if (L != p.max_prefix) {  // uniform over the workgroup
      dev::wait_vm<0>();  // the ring must be quiet before the same slots are filled again
      __syncthreads();
      n_spec = 0;
      set_range(L);
      n_rounds = (ts.t_end - ts.t_begin + TPR - 1) / TPR;
      if (PAGED) {
        ask_pages();
        dev::wait_vm<0>();
        fill_pages();
      }
    }
  }
  const int unit_id = b * n_kv_heads + kv;
  const bool has_tree = ts.t_end > ts.n_ptiles;
  if (PAGED && bad_page) __hip_atomic_fetch_or(p.err, kDevErrBadPage, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
  for (int r = 0; r < NR - 1; ++r)
    if (r >= n_spec && r < n_rounds) dma_round<D, NW, TPR, PAGED>(r, ts, lc, ring_addr + r * STAGE_BYTES);

  JK_TS(3);
  wait_dma<DMA_PER_ROUND>(n_rounds < NR - 1 ? n_rounds : NR - 1);  // (what is older than the first rounds)
  arrived_rows<kAskedRow>(q_raw);
  arrived<kAskedParent>(parent_lo);
  arrived<kAskedParent + 1>(parent_hi);
  dropped<kAskedLengths>(lengths);  // (more than 64 sequences have no use for it)
  dropped<kAskedLength>(L_one);
  // ---- ancestor sets (only workgroups that reach tree tiles need them); the barrier of the first round publishes them:
  // tree tiles are masked inside the loop only
  if (has_tree && wave == 0)
    build_ancestor_sets<kParamsAt>(lane, T, lane < T ? parent_lo : -1, lane + 64 < T ? parent_hi : -1, par_s, anc);

#pragma unroll
  for (int ks = 0; ks < DK; ++ks) {
    u32x4 v = q_raw[ks];
    if (!row_ok) v = u32x4{0u, 0u, 0u, 0u};
    st.q[ks] = __builtin_bit_cast(bf16x8, v);
  }
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) st.o[db][i] = 0.f;
  st.m = -INFINITY;
  st.l = 0.f;

  // mask of tile t: mode (see mask_tile), valid keys of a ragged prefix tile, visibility bits
  auto mask_of = [&](int t, int& mode, int& nvalid, unsigned int& bits) {
    mode = 0;
    nvalid = kTileKeys;
    bits = 0;
    if (t >= ts.t_end) {
      mode = 2;  // past the split: every key hidden (its LDS tile holds a copy of real data)
    } else if (t >= ts.n_ptiles) {
      const int tt = t - ts.n_ptiles;
      mode = 2;
      bits = (unsigned int)(anc[2 * my_node + (tt >> 1)] >> ((tt & 1) * 32));
    } else {
      nvalid = L - t * kTileKeys;
      mode = nvalid < kTileKeys ? 1 : 0;
    }
  };

  // ---- main loop.  Round r lives in ring slot r % NR; wave column wn takes tiles
  // (r*WN + wn)*KT .. +KT-1 of the split.  Before the barrier a wave waits for its own
  // transfers of round r; after the barrier every wave's have landed, and every wave has
  // finished round r-1, whose slot is therefore free for round r+NR-1.
  //
  // The pipelined pairs work in a fixed reference frame (see PairPipe).  If a score leaves it,
  // the wave says so in LDS after the loop, and the workgroup runs the loop once more, from
  // its first round, on the general path only (lazy rescale): rare, and the pairs stay free
  // of any conditional touch of the accumulators.
  bool left = false;     // a weight of this lane's row went beyond the frame (see PairPipe::reference)
  bool general = false;  // uniform: the repeat
  if (KT == 2 && tid == 0) *repeat_s = 0;  // (read behind the barrier that follows the loop)
  for (;;) {
  for (int r = 0; r < n_rounds; ++r) {
    // (what the round will do is worked out in front of the barrier: scalar arithmetic that
    // would otherwise stand between the barrier and the round's first LDS reads)
    const int tb = ts.t_begin + (r * WN + wn) * KT;
    const unsigned tile_a = ring_addr + (r % NR) * STAGE_BYTES + wn * KT * 2 * TILE_BYTES;  // K of the first tile
    const bool pair = KT == 2 && !general && (tb + 2) * kTileKeys <= L && tb + 2 <= ts.t_end;  // two full prefix tiles
    // the refill of the ring: on its own, or (full prefix tiles behind a pipelined pair)
    // piece by piece between the pair's MFMAs
    RoundPieces<D, NW, TPR> next;
    const int t_next = ts.t_begin + (r + NR - 1) * TPR;
    const bool refill = r + NR - 1 < n_rounds;
    // (paged caches refill in one go: with a base pointer per tile the interleaved refill measured slower)
    const bool spread = kSpread > 0 && !PAGED && WN == 1 && refill && pair && (t_next + TPR) * kTileKeys <= L;
    next.tile_elems = (long long)kTileKeys * ts.kc_sl;
    next.base = lc.cache + (long long)t_next * next.tile_elems;
    next.slot = ring_addr + ((r + NR - 1) % NR) * STAGE_BYTES;
    next.lc = &lc;
    const int ahead = n_rounds - 1 - r;  // rounds issued after r: min(NR-2, ahead)
    wait_dma<DMA_PER_ROUND>(ahead < NR - 2 ? ahead : NR - 2);
    __syncthreads();
    if (r == 0) JK_TS(4);
    if (refill && !spread) dma_round<D, NW, TPR, PAGED>(r + NR - 1, ts, lc, ring_addr + ((r + NR - 1) % NR) * STAGE_BYTES);
    if (pair && spread) {
      PairPipe<D>::template run<kSpread>(st, tile_a + k_lane, tile_a + TILE_BYTES + v_lane, scale_log2, next, r == 0);
    } else if (pair) {
      PairPipe<D>::template run<0>(st, tile_a + k_lane, tile_a + TILE_BYTES + v_lane, scale_log2, next, r == 0);
    } else if (KT == 2 && WN == 1 && !general && tb + 1 == ts.t_end && (tb + 1) * kTileKeys <= L) {
      lone_tile<D>(st, tile_a + k_lane, tile_a + TILE_BYTES + v_lane, scale_log2, r == 0);  // no mask, half the work
    } else if (tb < ts.t_end) {
      int mode, nvalid;
      unsigned int bits;
      floatx16 s0, s1;
      // (the general path may rescale the sums: what the fast paths left in them is tested first)
      if (KT == 2 && !general) left = left || PairPipe<D>::left_frame(st);
      qk_tiles<D, KT>(st, tile_a + k_lane, s0, s1);
      mask_of(tb, mode, nvalid, bits);
      mask_tile(s0, mode, nvalid, bits, g);
      if (KT == 2) {
        mask_of(tb + 1, mode, nvalid, bits);
        mask_tile(s1, mode, nvalid, bits, g);
      }
      softmax_pv<D, KT>(st, s0, s1, tile_a + TILE_BYTES + v_lane, scale_log2);
    }
  }
  if (KT == 2 && !general && (left || PairPipe<D>::left_frame(st))) *repeat_s = 1;
  JK_TS(5);
  if (KT != 2) break;
  __syncthreads();  // every wave is done with the ring before it is filled again
  if (general || __builtin_amdgcn_readfirstlane(*repeat_s) == 0) break;
  general = true;
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) st.o[db][i] = 0.f;
  st.m = -INFINITY;
  st.l = 0.f;
#pragma unroll
  for (int r = 0; r < NR - 1; ++r)
    if (r < n_rounds) dma_round<D, NW, TPR, PAGED>(r, ts, lc, ring_addr + r * STAGE_BYTES);
  }

  // ---- epilogue.  A wave of a single key column owns the result of its 32 rows.  Two key columns share theirs: column
  // wn finishes the half of the columns that its first accumulators hold (see v_lane), parks the other half and its
  // (max, sum) in LDS for the other column's wave of the same rows, and folds what that one parked for it into its own,
  // register for register (all waves share one layout, so a lane reads what its double wrote: consecutive 16 bytes a
  // lane, no bank conflict).  They park in the ring slot of the last round but one, which every wave left before the last
  // round's barrier.  This part is bound by the instructions of a lone wave per SIMD: with column 0 folding and storing
  // whole rows behind column 1's a layer of a 7B model of 1024 keys took 10.1 us and takes 9.8, eleven sequences of 120
  // keys (8 heads, six nodes, undivided) 7.5 and 7.1, two of 377 keys in two splits 8.9 and 8.4.
  // Lane (row, g) holds, per 32-wide block db and quarter q4, the 4 columns 32*db + 8*q4 + 4*g .. +3 of its row.
  // (the lane's indices are worked out afresh, from the execution mask: kept in registers
  // across the tile loop, which has none to spare, they - or the thread id they come from -
  // are spilled to memory and read back here)
  constexpr int OB = P_::OB, OCOLS = P_::OCOLS;  // 32-wide blocks, and columns, that a wave finishes
  const int lane_e = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  const int c32_e = lane_e & 31, g_e = lane_e >> 5;
  const bool whole = MERGE == 0 && splits == 1;  // the final result, not a split's partial
  float mx = st.m, lsum = half_swap_sum(st.l);
  unsigned char* slots = smem + (WN == 2 ? ((n_rounds + NR - 2) % NR) * STAGE_BYTES : 0);
  unsigned char* patch = slots + wave * P_::SLOT_BYTES;
  if constexpr (WN == 2) {
    const int partner = wave ^ WM;  // the same rows' wave of the other column
    float4* park = reinterpret_cast<float4*>(slots + partner * P_::SLOT_BYTES) + lane_e;
#pragma unroll
    for (int db = 0; db < OB; ++db)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const floatx16& o = st.o[OB + db];
        park[(db * 4 + q4) * 64] = make_float4(o[4 * q4], o[4 * q4 + 1], o[4 * q4 + 2], o[4 * q4 + 3]);
      }
    mlbuf[wave * kWaveRows + c32_e] = make_float2(mx, lsum);  // (both halves of the wave hold the row's)
    __syncthreads();
    const float2 ml = mlbuf[partner * kWaveRows + c32_e];
    const float m_all = fmaxf(mx, ml.x);
    const float m_use = (m_all == -INFINITY) ? 0.f : m_all;
    float w0 = fast_exp2(mx - m_use), w1 = fast_exp2(ml.x - m_use);
    lsum = fmaf(ml.y, w1, lsum * w0);
    mx = m_all;
    if (whole) {  // lsum > 0: every row sees at least its own tree key
      w0 /= lsum;
      w1 /= lsum;
    }
    const float4* parked = reinterpret_cast<const float4*>(patch) + lane_e;
#pragma unroll
    for (int db = 0; db < OB; ++db)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const float4 v = parked[(db * 4 + q4) * 64];
        floatx16& o = st.o[db];
        o[4 * q4] = fmaf(v.x, w1, o[4 * q4] * w0);
        o[4 * q4 + 1] = fmaf(v.y, w1, o[4 * q4 + 1] * w0);
        o[4 * q4 + 2] = fmaf(v.z, w1, o[4 * q4 + 2] * w0);
        o[4 * q4 + 3] = fmaf(v.w, w1, o[4 * q4 + 3] * w0);
      }
  } else if (whole) {
    const float mul = 1.f / lsum;
#pragma unroll
    for (int db = 0; db < OB; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) st.o[db][i] *= mul;
  }
  JK_TS(6);
  // ---- store: the final result (no splits) or the split's partial, in fp32 or in bf16 (AttnPlan::fine; the running max and
  // sum are always fp32).
  // (a lone wave per SIMD issues an instruction every five to eight cycles: this part of the
  // kernel is bound by its instruction count, hence the uniform branches around whole loops
  // rather than conditions inside them)
  const long long prow0 = ((long long)unit_id * splits + split) * p.m_pad + qtile * QROWS + wm * kWaveRows;
  const int rows_valid = M - (qtile * QROWS + wm * kWaveRows);  // rows of this wave that exist (32 or more: all)
  if (!whole && wn == 0 && c32_e < rows_valid && g_e == 0) {
    if (p.through & 2) dev::store_through(p.part_ml + prow0 + c32_e, dev::store_u32x2{__float_as_uint(mx), __float_as_uint(lsum)});
    else p.part_ml[prow0 + c32_e] = make_float2(mx, lsum);
  }
  const bool thr = MERGE == 0 && (p.through & 1);
  constexpr int LD = P_::PATCH_LD, LPR = OCOLS / 8, RPI = 64 / LPR;  // bytes a patch row, lanes a row, rows a store
  const int chunk = lane_e % LPR, rsub = lane_e / LPR;
  const unsigned char* src0 = patch + rsub * LD + chunk * 16;
  if (FINE || (MERGE == 0 && !whole && (p.through & 4))) {
    if constexpr (WN == 2) {
      // a block of 32 columns at a time by way of the patch (see below): 128-byte rows, their 16-byte chunks swizzled by the
      // row.  (Straight from the accumulators, 32 bytes into each of 32 rows a store, four sequences of 400 keys, 8B, took 12.8
      // us instead of 12.2.)
      typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
      const unsigned prow = (unsigned)(size_t)LDS_PTR(unsigned char, patch) + c32_e * 128 + ((g_e ^ (c32_e & 7)) << 4);
      const int r8 = lane_e / 8, c8 = lane_e % 8;
      const unsigned char* from = patch + r8 * 128 + ((c8 ^ r8) << 4);
      float* dst0 = reinterpret_cast<float*>(p.part_o) + (prow0 + r8) * D + wn * OCOLS + c8 * 4;
#pragma unroll
      for (int db = 0; db < OB; ++db) {
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const floatx16& o = st.o[db];
          *(lds_u32x4*)(size_t)(prow ^ (q4 << 5)) = u32x4{__float_as_uint(o[4 * q4]), __float_as_uint(o[4 * q4 + 1]),
                                                          __float_as_uint(o[4 * q4 + 2]), __float_as_uint(o[4 * q4 + 3])};
        }
        u32x4 v[kWaveRows / 8];
#pragma unroll
        for (int k = 0; k < kWaveRows / 8; ++k) v[k] = *reinterpret_cast<const u32x4*>(from + k * 1024);
#pragma unroll
        for (int k = 0; k < kWaveRows / 8; ++k) {
          asm volatile("" : "+v"(v[k]));  // (read outside the condition)
          if (k * 8 < rows_valid) {
            if (thr) dev::store_through(dst0 + k * 8 * D + 32 * db, v[k]);
            else *reinterpret_cast<u32x4*>(dst0 + k * 8 * D + 32 * db) = v[k];
          }
        }
      }
    } else {
      // half of the columns at a time by way of the patch (see below), as many bytes a row as all of them in bf16
      unsigned char* prow = patch + c32_e * LD + g_e * 16;
      unsigned char* dst0 = reinterpret_cast<unsigned char*>(p.part_o) + ((prow0 + rsub) * D + chunk * 4) * 4;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int db = 0; db < DB / 2; ++db)
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) {
            const floatx16& o = st.o[h * (DB / 2) + db];
            *reinterpret_cast<float4*>(prow + (32 * db + 8 * q4) * 4) = make_float4(o[4 * q4], o[4 * q4 + 1], o[4 * q4 + 2], o[4 * q4 + 3]);
          }
        u32x4 v[kWaveRows / RPI];
#pragma unroll
        for (int k = 0; k < kWaveRows / RPI; ++k) v[k] = *reinterpret_cast<const u32x4*>(src0 + k * RPI * LD);
#pragma unroll
        for (int k = 0; k < kWaveRows / RPI; ++k) {
          unsigned char* dst = dst0 + k * RPI * D * 4 + h * D * 2;
          asm volatile("" : "+v"(v[k]));
          if (k * RPI < rows_valid) {
            if (thr) dev::store_through(dst, v[k]);
            else *reinterpret_cast<u32x4*>(dst) = v[k];
          }
        }
      }
    }
  } else {
    // bf16: the accumulator layout gives a lane 4 columns here and 4 there of one row, 8 bytes each.  So the wave
    // first lays its 32 rows out in LDS (where its partner's share was parked: LDS operations of a wave complete in
    // order) and reads them back row-wise, and a store covers whole lines of a few rows.
    unsigned char* prow = patch + c32_e * LD + g_e * 8;
#pragma unroll
    for (int db = 0; db < OB; ++db)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        bf16x2 lo, hi;
        lo[0] = (__bf16)st.o[db][4 * q4];
        lo[1] = (__bf16)st.o[db][4 * q4 + 1];
        hi[0] = (__bf16)st.o[db][4 * q4 + 2];
        hi[1] = (__bf16)st.o[db][4 * q4 + 3];
        uint2 pk;
        pk.x = __builtin_bit_cast(unsigned int, lo);
        pk.y = __builtin_bit_cast(unsigned int, hi);
        *reinterpret_cast<uint2*>(prow + (32 * db + 8 * q4) * 2) = pk;
      }
    u32x4 v[kWaveRows / RPI];
#pragma unroll
    for (int k = 0; k < kWaveRows / RPI; ++k) v[k] = *reinterpret_cast<const u32x4*>(src0 + k * RPI * LD);
    // (all read in front of the first store and its condition: read and stored one after the other, a trip to LDS each, the
    // waves whose rows end among their 32 kept their row tile's merge waiting)
    if (whole) {
#pragma unroll
      for (int k = 0; k < kWaveRows / RPI; ++k) {
        const int rr = k * RPI + rsub;                               // row of the wave
        const int m = qtile * QROWS + wm * kWaveRows + rr;           // query row
        asm volatile("" : "+v"(v[k]));
        if (rr < rows_valid) {
          const int node = div_mg(m, p.mg_g);
          uint16_t* dst = p.out + b * p.o_sb + node * p.o_st + (long long)(kv * G + (m - node * G)) * p.o_sh + wn * OCOLS + chunk * 8;
          if (thr) dev::store_through(dst, v[k]);
          else *reinterpret_cast<u32x4*>(dst) = v[k];
        }
      }
    } else {
      // partial rows are D elements apart: one address, constant steps; what a store holds besides rows that exist goes to
      // the padding of their row tile, which nobody reads
      unsigned char* dst0 = reinterpret_cast<unsigned char*>(p.part_o) + ((prow0 + rsub) * D + wn * OCOLS + chunk * 8) * 2;
      auto store_rows = [&](auto through) {
#pragma unroll
        for (int k = 0; k < kWaveRows / RPI; ++k) {
          asm volatile("" : "+v"(v[k]));
          if (k * RPI >= rows_valid) break;  // (uniform)
          if (decltype(through)::value) dev::store_through(dst0 + k * RPI * D * 2, v[k]);
          else *reinterpret_cast<u32x4*>(dst0 + k * RPI * D * 2) = v[k];
        }
      };
      if (thr) store_rows(std::true_type{});
      else store_rows(std::false_type{});
    }
  }
  if constexpr (MERGE > 0) {
    // ---- merge of the group's splits in this kernel.  Every workgroup of the group owns the slice
    // of R = ceil(QROWS / splits) rows numbered like its split and merges it once all partials are
    // in L2.  Waiting is bounded: a workgroup that gives up records its slice in the group's mask
    // and leaves; the group's last arriver, which never waits, then merges those slices as well,
    // so the result is complete whenever every workgroup of the group runs, however late.
    // (The arguments this part needs are fetched from the kernel-argument segment here rather than
    // held in scalar registers across the tile loop, which has none to spare.)
    typedef __attribute__((address_space(4))) const KParams KArgs;
    KArgs* late = (KArgs*)((__attribute__((address_space(4))) const char*)__builtin_amdgcn_kernarg_segment_ptr() + kParamsAt);
    asm volatile("" : "+s"(late));
    const int tid_e = wave * 64 + lane_e;  // (the thread id, rebuilt: see the note on lane_e above)
    {
      int* mode_s = repeat_s + 1;  // 0 leave, 1 merge own slice, 2 also the slices in mode_s[1..2]
      // (what the merge of this workgroup's own slice needs besides the partials: computed now, while
      // the partial stores travel and before the wait for the group)
      MergeArgs ma;
      ma.part_o = late->part_o; ma.part_ml = late->part_ml; ma.out = late->out;
      ma.M = late->M; ma.m_pad = late->m_pad; ma.splits = late->splits; ma.G = late->G; ma.mg_g = late->mg_g;
      ma.o_sb = late->o_sb; ma.o_st = late->o_st; ma.o_sh = late->o_sh;
      const int slice_rows = late->merge_rows, merge_shift = MERGE < 6 ? tva::merge_shift_of(MERGE) : late->merge_shift;
      const int tile_row0 = qtile * QROWS;
      MergeThread mt = merge_prepare<D, THREADS, QROWS, FINE>(ma, unit_id, b, kv, split, slice_rows, merge_shift, tile_row0, tid_e);
      unsigned* word = late->sync + group_word(unit_id * late->n_qtiles + qtile);
      unsigned limit = late->spin_limit;
      // (here, and not where it is used: left alone, the compiler puts it behind the wait for the group)
      int live = mt.live_a;
      asm volatile("" : "+v"(mt.raw_off), "+v"(mt.ml_off), "+v"(mt.dst_off), "+v"(mt.r_b), "+v"(live), "+s"(mt.unit_end), "+s"(mt.row_lo), "+s"(mt.row_hi));
      asm volatile("" : "+s"(word), "+s"(limit));
      mt.live_a = live != 0;
      JK_TS(7);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's partial stores have reached L2
      __syncthreads();
      JK_TS(8);
      if (tid_e == 0) {
        const unsigned S = (unsigned)splits;
        const unsigned old = l2_atomic_add(word, 1u);
        const unsigned epoch = old >> 16;
        int mode = 1;
        unsigned m_lo = 0u, m_hi = 0u;
        if ((old & kSyncCountMask) == S - 1) {
          const unsigned gave_up = (old >> 8) & 0xffu;
          l2_atomic_add_noret(word, kSyncEpochOne - S - gave_up * kSyncGaveUpOne);
          if (gave_up) {
            mode = 2;
            m_lo = l2_atomic_swap(word + 1, 0u);
            m_hi = l2_atomic_swap(word + 2, 0u);
          }
        } else if (mt.row_lo >= min(mt.row_hi, late->M - tile_row0)) {
          mode = 0;  // (no row of the slice exists: nothing to wait for, and the CU is free for the next workgroup)
        } else {
          unsigned polls = 0;
          for (;;) {
            const unsigned v = l2_atomic_add(word, 0u);
            if ((v >> 16) != epoch || (v & kSyncCountMask) == S) break;
            if (++polls > limit) {
              l2_atomic_or(word + 1 + (split >> 5), 1u << (split & 31));
              const unsigned v2 = l2_atomic_add(word, kSyncGaveUpOne);
              // (complete after all, between the last poll and the mark: the last arriver has not seen
              // the mark, so this slice is still ours; the stray mark only costs a later call a repeat)
              if (!((v2 >> 16) != epoch || (v2 & kSyncCountMask) == S)) mode = 0;
              __hip_atomic_fetch_or(late->err, kDevErrMergeWait, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              break;
            }
            __builtin_amdgcn_s_sleep(1);
          }
        }
        mode_s[0] = mode;
        mode_s[1] = (int)m_lo;
        mode_s[2] = (int)m_hi;
      }
      __syncthreads();
      JK_TS(9);
      const int mode = __builtin_amdgcn_readfirstlane(mode_s[0]);
      if (mode != 0) {
        // (No line of the partials can sit in this CU's vector cache: the cache starts every kernel
        // empty, this kernel reads partials nowhere else, and no partial is rewritten after the group
        // is complete.  The loads below therefore go to L2 without an invalidate in front of them.)
        asm volatile("" ::: "memory");
        float* wbuf = reinterpret_cast<float*>(smem);  // (ring and epilogue buffers are dead: every wave is past its stores)
        unsigned long long left_over = 0ull;  // the slices of workgroups that gave up waiting
        if (mode == 2)
          left_over = ((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane(mode_s[2]) << 32) |
                      (unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane(mode_s[1]);
        left_over &= ~(1ull << split);
        for (;;) {
          if (mt.row_lo < mt.row_hi) {  // (uniform)
            merge_rows<D, THREADS, QROWS, tva::merge_shift_of(MERGE), FINE>(ma, mt, merge_shift, b, kv, tile_row0, tid_e, wbuf);
            __syncthreads();  // wbuf is free again
          }
          if (left_over == 0ull) break;
          const int j = __ffsll((long long)left_over) - 1;
          left_over &= left_over - 1ull;
          mt = merge_prepare<D, THREADS, QROWS, FINE>(ma, unit_id, b, kv, j, slice_rows, merge_shift, tile_row0, tid_e);
        }
      }
    }
  }
#ifdef JK_TIMING
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (so that the last stamp includes the result stores)
#endif
  JK_TS(10);
}

template <int D, int WM, int WN, int KT, bool PAGED, bool DEEP>
hipError_t launch_one(const KParams& kp, hipStream_t stream) {
  using P_ = Plan<D, WM, WN, KT, PAGED, DEEP>;
  auto kern = tva_bf16_kernel<D, WM, WN, KT, PAGED, DEEP, JK_MERGE>;
  static LdsLimitRaised raised;
  if (hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(kern), P_::SMEM, raised); e != hipSuccess) return e;
  return launch_kernel(kern, dim3(kp.total_wgs), dim3(P_::THREADS), P_::SMEM, stream, kp.prefix_len, kp.B, kp.total_wgs, kp.n_qtiles, kp.splits, kp.units_per_xcd,
                     kp.second_turn, kp.Hkv, (unsigned)kp.mg_qtiles, (unsigned)kp.mg_splits, (unsigned)kp.mg_hkv, (unsigned)kp.mg_upx, kp);
}
template <int D, bool PAGED>
hipError_t launch_arranged(const KParams& kp, const AttnPlan& pl, hipStream_t stream) {
  if (pl.wm == 4 && pl.wn == 1 && pl.kt == 2) return launch_one<D, 4, 1, 2, PAGED, false>(kp, stream);
  if (pl.wm == 2 && pl.wn == 2 && pl.kt == 1)
    return pl.deep ? launch_one<D, 2, 2, 1, PAGED, true>(kp, stream) : launch_one<D, 2, 2, 1, PAGED, false>(kp, stream);
  return hipErrorInvalidValue;
}

}  // namespace

#ifdef JK_TIMING
#define JK_CAT2(a, b) a##b
#define JK_CAT(a, b) JK_CAT2(a, b)
extern "C" int JK_CAT(jk_debug_read_timing, JK_MERGE)(unsigned long long* host, size_t n) {
  return (int)hipMemcpyFromSymbol(host, HIP_SYMBOL(g_jk_ts), n * sizeof(unsigned long long));
}
#endif

namespace tva {
template <>
hipError_t launch_merged<JK_MERGE>(const KParams& kp, int head_dim, const AttnPlan& pl, hipStream_t stream) {
  const bool paged = kp.block_table != nullptr;
  if (head_dim == 128) return paged ? launch_arranged<128, true>(kp, pl, stream) : launch_arranged<128, false>(kp, pl, stream);
  if (head_dim == 64) return paged ? launch_arranged<64, true>(kp, pl, stream) : launch_arranged<64, false>(kp, pl, stream);
  return hipErrorInvalidValue;
}
}  // namespace tva

#if JK_MERGE == 0
hipError_t launch_tva_bf16(const AttnArgs& a, const AttnPlan& pl, hipStream_t stream) {
  KParams kp;
  kp.q = static_cast<const uint16_t*>(a.q);
  kp.kc = static_cast<const uint16_t*>(a.k_cache);
  kp.vc = static_cast<const uint16_t*>(a.v_cache);
  kp.kt = static_cast<const uint16_t*>(a.k_tree);
  kp.vt = static_cast<const uint16_t*>(a.v_tree);
  kp.parent = a.parent;
  kp.prefix_len = a.prefix_len;
  kp.out = static_cast<uint16_t*>(a.out);
  kp.part_o = a.part_o;
  kp.part_ml = a.part_ml;
  const jk_attn_desc& d = a.d;
  kp.B = d.batch; kp.T = d.n_tree; kp.Hkv = d.n_kv_heads; kp.G = d.n_q_heads / d.n_kv_heads;
  kp.M = pl.m_rows; kp.m_pad = pl.m_pad; kp.max_prefix = a.max_prefix_len;
  kp.splits = pl.splits; kp.n_qtiles = pl.n_qtiles;
  const long long work = (long long)d.batch * d.n_kv_heads * pl.splits * pl.n_qtiles;
  kp.total_wgs = (int)((work + 7) / 8 * 8);
  kp.q_sb = d.q_stride_b; kp.q_st = d.q_stride_t; kp.q_sh = d.q_stride_h;
  kp.kc_sb = d.kc_stride_b; kp.kc_sl = d.kc_stride_l; kp.kc_sh = d.kc_stride_h;
  kp.kt_sb = d.kt_stride_b; kp.kt_st = d.kt_stride_t; kp.kt_sh = d.kt_stride_h;
  kp.o_sb = d.o_stride_b; kp.o_st = d.o_stride_t; kp.o_sh = d.o_stride_h;
  kp.scale_log2 = a.scale_log2;
  auto magic = [](int d) { return (1ull << 32) / (unsigned long long)d + 1ull; };
  kp.mg_qtiles = magic(pl.n_qtiles);
  kp.mg_splits = magic(pl.splits);
  kp.mg_splits_m1 = magic(pl.splits > 1 ? pl.splits - 1 : 1);
  kp.mg_hkv = magic(d.n_kv_heads);
  kp.mg_g = magic(kp.G);

  kp.block_table = a.block_table;
  kp.max_blocks = a.max_blocks;
  kp.n_pages = a.n_pages;
  kp.tpp = a.block_table ? a.page_size / kTileKeys : 1;
  kp.page_stride = a.page_stride;
  kp.mg_tpp = magic(kp.tpp);
  // Results written with ordinary stores stay dirty in the XCDs' L2s until the end of the
  // kernel writes them back.  When the whole grid is resident at once (every workgroup ends
  // within the same microsecond) that write-back is exposed, and stores that go through to
  // memory at once measured faster (c3 -0.2 us, c2 -0.65 us per call); with several
  // workgroups per CU in turn, dirty lines of finished workgroups drain while the others
  // compute, and ordinary stores measured faster (c4 +0.8 us with write-through).  The small
  // (max, sum) pairs: through only for the 2x2 arrangement (c2 -0.35 us; c3, 4x1: +0.25 us).
  const bool one_wave = work <= (long long)device_cu_count();
  kp.through = (one_wave ? 1 : 0) | (one_wave && pl.wn > 1 ? 2 : 0);
  // merged in the kernel: ordinary stores (measured: the L2 passes them on and keeps no line of them, but they are
  // acknowledged after 0.7 us and read back in 0.4; stores through to memory take 1.3 and 1.0)
  const bool fused = pl.fused && pl.splits > 1;
  if (fused && pl.wm != 8) kp.through = 0;
  if (pl.fine) kp.through |= 4;
  if (fused && pl.wm != 8 && (pl.fine != 0) != (pl.splits <= 3)) return hipErrorInvalidValue;  // (what the instances assume)
  kp.sync = a.sync;
  // (a lane per sequence in the ranking; the XCDs get whole units)
  const long long units = (long long)d.batch * d.n_kv_heads;
  const bool ranked = pl.ranked != 0;
  const int per_xcd_units = units >= 8 ? (int)(units / 8) : 1;  // (tva_wide.hip only asks whether there are any)
  kp.units_per_xcd = ranked ? per_xcd_units : 0;
  kp.mg_upx = magic(per_xcd_units);
  const int xcd_cus = device_cu_count() / 8, per_xcd = kp.total_wgs / 8;
  kp.second_turn = ranked && per_xcd > xcd_cus && per_xcd <= 2 * xcd_cus ? xcd_cus : kp.total_wgs;
  kp.err = a.err;
  kp.spin_limit = tuning().spin_limit >= 0 ? (unsigned)tuning().spin_limit : 4096u;  // about 2 ms of polling here, 1 ms in tva_wide.hip
  kp.merge_rows = (pl.q_rows + pl.splits - 1) / pl.splits;
  kp.merge_shift = 0;
  while ((1 << kp.merge_shift) < pl.splits) ++kp.merge_shift;
  if (pl.wm == 8) return tva::launch_wide(kp, d.head_dim, stream);
  if (pl.wm == 1) return tva::launch_direct(kp, d.head_dim, stream);
  switch (fused ? tva::merge_of(pl.splits) : 0) {
    case 0: return tva::launch_merged<0>(kp, d.head_dim, pl, stream);
    case 1: return tva::launch_merged<1>(kp, d.head_dim, pl, stream);
    case 2: return tva::launch_merged<2>(kp, d.head_dim, pl, stream);
    case 3: return tva::launch_merged<3>(kp, d.head_dim, pl, stream);
    case 4: return tva::launch_merged<4>(kp, d.head_dim, pl, stream);
    case 5: return tva::launch_merged<5>(kp, d.head_dim, pl, stream);
    default: return tva::launch_merged<6>(kp, d.head_dim, pl, stream);
  }
}
#endif

}  // namespace jk
