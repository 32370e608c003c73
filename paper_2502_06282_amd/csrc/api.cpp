// C-ABI entry points of libjakiro_verify: argument checks, launch planning,
// kernel launches.  No device memory is allocated here and nothing synchronises.
#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <initializer_list>
#include <random>

#include "jk_divide.h"
#include "jk_internal.h"

namespace jk {

int device_cu_count() {
  static int cus = 0;  // same value whoever writes it first
  if (cus == 0) {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
      cus = n;
    else
      cus = 256;
  }
  return cus;
}

// A word that no launch of this process had before (up to 2^47 launches) and that memory is not likely
// to hold
unsigned long long meeting_tag() {
  static const unsigned long long seed = [] {
    std::random_device r;
    return ((unsigned long long)r() << 32) | r();
  }();
  static std::atomic<unsigned long long> count{0};
  // (a bijection of 47 bits: odd multiplications and shifts to the right)
  unsigned long long v = (seed + count.fetch_add(1, std::memory_order_relaxed)) & 0x7FFFFFFFFFFFull;
  v = (v * 0x9E3779B97F4Bull) & 0x7FFFFFFFFFFFull;
  v ^= v >> 23;
  v = (v * 0xC2B2AE3D27D5ull) & 0x7FFFFFFFFFFFull;
  return ((v ^ (v >> 25)) << 16) | (1ull << 63);
}

namespace {
int env_int(const char* name, int fallback) {
  const char* e = std::getenv(name);
  return e && *e ? std::atoi(e) : fallback;
}
Tuning tuning_from_env() {
  Tuning t;
  t.attn_wm = env_int("JK_ATTN_WM", 0);
  t.attn_wn = env_int("JK_ATTN_WN", 0);
  t.attn_splits = env_int("JK_ATTN_SPLITS", 0);
  t.attn_fused = env_int("JK_ATTN_FUSED", -1);
  t.attn_deep = env_int("JK_ATTN_DEEP", -1);
  t.accept_single = env_int("JK_ACCEPT_SINGLE", 0);
  t.spin_limit = env_int("JK_SPIN_LIMIT", -1);
  t.ring_gemm = env_int("JK_RING_GEMM", -1);
  t.narrow_gemm = env_int("JK_NARROW_GEMM", -1);
  t.verbose = env_int("JK_ATTN_VERBOSE", 0);
  return t;
}
}  // namespace

Tuning& tuning() {
  static Tuning t = tuning_from_env();  // the environment is read once, here
  return t;
}

namespace {
constexpr int kMaxDevices = 64;
int g_xcd_state[kMaxDevices];  // per device: 0 not checked (jk_init not called), 1 round-robin verified, 2 not round-robin
}  // namespace

bool xcd_placement_verified() {
  int dev = -1;
  return hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < kMaxDevices && g_xcd_state[dev] == 1;
}

namespace {
bool desc_ok(const jk_attn_desc& d) {
  if (d.batch < 1 || d.n_tree < 1 || d.n_tree > JK_MAX_TREE) return false;
  if (d.n_q_heads < 1 || d.n_kv_heads < 1 || d.n_q_heads % d.n_kv_heads) return false;
  if (d.dtype != JK_BF16 && d.dtype != JK_F32) return false;
  if (!(d.scale >= 0.f) || !std::isfinite(d.scale)) return false;
  return true;
}
bool shape_supported(const jk_attn_desc& d) {
  if (d.dtype == JK_BF16) return d.head_dim == 64 || d.head_dim == 128;
  return d.head_dim >= 4 && d.head_dim <= 256 && d.head_dim % 4 == 0;
}
}  // namespace

// Constants of the attention plan's time estimate, fitted together to timed plans of drawn shapes (those timings were not
// kept).  What they are worth is measured by profiles/attention_plan_times.py: over the 1000 shapes and 11711 plans of
// profiles/attention_plan_times.csv (batch 1 - 32, 1 - 128 tree nodes, 2 - 40 KV heads, head_dim 64/128, prefixes up to
// 32k) the plan the estimate takes is 1.3 % slower than the best one timed (geometric mean; 5 % at the 90th percentile,
// 17 % at the 99th); runs of one plan differ by about 1 %.  The fit is of the whole estimate: single constants are near,
// not at, what a part takes when it is timed alone.
struct PlanModel {
  double round_4x1 = 1.13, round_4x1_d64 = 0.84;  // us per round (a pair of 32-key tiles) of a 4x1 workgroup alone on its CU
  double round_2x2 = 0.90, round_2x2_d64 = 0.58;  // us per round (one tile per key column) of a 2x2 workgroup
  double tail_2x2 = 1.03;       // a ragged or tree tile costs this much of a round on top, shared by the splits
  double share_4x1 = 1.45, share_2x2 = 1.37;      // two workgroups on a CU take this many times one's time
  double far_bytes = 9.0e7;     // K/V beyond this come from HBM, not from a cache: the longer latency shows with
  double far_2x2 = 1.24, far_2x2_shared = 1.11, far_deep = 1.02;  // the 2x2 arrangement's one round in flight
  double stream = 7.0e6;        // bytes per us all CUs together
  double startup = 5.7;         // us of a call outside its rounds: launch, first K/V data (2.6 - 2.8 us after it), epilogue
  double startup_4x1 = 1.03;    // (more for twice the rows)
  double turn_0 = 0.35, turn_step = 0.14, turn_min = 0.02;  // how much of a last, partly filled turn of two workgroups per CU
                                // shows: a third after one full turn, less with each further one (they drift apart)
  double merge_fused_fixed = 1.63, merge_fused_per_mb = 0.30;  // merge inside the kernel
  double merge_kernel_fixed = 2.1, merge_kernel_per_mb = 0.36; // second launch
  double merge_16 = 1.4;        // either way, for each 16 splits beyond the first (their loads go out in turns)
  // 256 rows per workgroup (tva_wide.hip), one of them per CU: us per tile without a mask, per other tile (the first, tree
  // and ragged ones, those that four does not divide), per turn of workgroups, per call, per level of the pairwise merge
  // and per MB that changes hands there.  (Searched together like the others; a tile takes 0.55 us timed alone.  The plan takes
  // this kernel for 72 of the 1000 shapes above, and it is the fastest for 67; over the 72 the best plan of the other
  // kernels is 1.11 times as slow in the geometric mean, 0.88 to 1.31.)
  double wide_tile = 0.44, wide_tile_d64 = 0.385, wide_slow = 1.06, wide_slow_d64 = 0.70;
  double wide_hot = 0.31, wide_hot_tiles = 500.0;  // the clock falls under the matrix units' load: the tiles of a long call
                                // take up to this much longer
  double wide_stream = 1.0e7, wide_turn = 5.3, wide_call = 2.8, wide_level = 2.0, wide_merge_per_mb = 0.57;
  double wide_margin = 1.02;    // (near ties go to the others)
  // 16 rows per workgroup and K, V in registers (tva_direct.hip): us of a call outside its blocks, per turn of four blocks of 32
  // keys, per workgroup of a CU beyond the first, for trees of more than 64 nodes (their ancestors); bytes per us that a CU
  // draws of K and V, and all CUs together.  Fitted to the times of 320 drawn calls of up to 1300 keys of prefix and 2000
  // workgroups (5.0 % rms; those timings were not kept).  The others' estimates of such short calls are 1.2 times what they take (2x2
  // waves, geometric mean): direct_level puts this one beside them.  (At 1.3 the 320 calls take 0.840 of what they take without
  // this kernel, the best choice would take 0.834, and three are slower than without it by more than 3 %, 7 % at most; at 1.2 ten
  // are, at 1.4 they take 0.849.)  The plan takes it for 273 of the 1000 shapes above, and it is the fastest for 291; over the 273 the
  // best plan of the other kernels is 1.31 times as slow, 0.92 to 1.62 (two are slower with it by more than 3 %: 38 and 145 MB
  // of K and V, 8 and 6 %).
  double direct_call = 3.31, direct_call_d64 = 2.97, direct_round = 0.66, direct_round_d64 = 0.63, direct_next = 0.81,
         direct_deep_tree = 0.65, direct_draw = 6.05e4, direct_stream = 3.40e7, direct_level = 1.3;
};

namespace {
// Whether a workspace has room for fp32 ranges in parts; the line from which they are taken so: see compute_attn_plan
bool f32_in_parts(long long keys, int head_dim) { return keys >= (head_dim <= 64 ? 300 : head_dim <= 128 ? 200 : 112); }

// A workspace serves every call that is no larger in batch, nodes, heads, head_dim and prefix bound than the one it was
// sized for.  Partial results alone do not have that order - a smaller call may be cut into more splits, and take more
// room - so a plan's partial rows stay below a bound that grows with each of those numbers, and the size query answers
// with the bound.  bf16: as many splits as the keys allow, but no more than ten full turns of the widest workgroups
// (kTurns; 84 MB at head_dim 128) unless that is less than kEach results per query row: 38 of 120000 plans of drawn
// shapes would be cut into more (at eight turns and four results 250, at six 962).
size_t most_part_rows(const jk_attn_desc& d, int max_prefix_len) {  // over all (sequence, KV head) units
  constexpr long long kTurns = 10, kEach = 3;
  const long long units = (long long)d.batch * d.n_kv_heads, m = (long long)d.n_tree * (d.n_q_heads / d.n_kv_heads);
  const long long cus = device_cu_count();
  auto least = [](long long a, long long b) { return a < b ? a : b; };
  auto most = [](long long a, long long b) { return a > b ? a : b; };
  if (d.dtype == JK_BF16) {
    const long long n_tiles = (max_prefix_len + kTileKeys - 1) / kTileKeys + (d.n_tree + kTileKeys - 1) / kTileKeys;
    const long long s_min = (n_tiles + kMaxTilesPerSplit - 1) / kMaxTilesPerSplit;
    const long long s_top = least(most(n_tiles / 4, s_min), kMaxSplits);  // (at least two rounds of two tiles per split)
    if (s_top <= 1) return 0;
    const long long base = units * ((m + 127) / 128 * 128);
    return (size_t)least(base * s_top, most(kTurns * cus * 128, base * most(kEach, s_min)));
  }
  // fp32: a result per range of 1024 keys, or, where workgroups of sixteen rows are fewer than CUs, up to eight of it
  const long long keys = (long long)max_prefix_len + d.n_tree, s = (keys + 1023) / 1024;
  const long long whole = s > 1 ? units * m * s : 0, divided = f32_in_parts(keys, d.head_dim) ? least(16 * cus, units * m * least(8 * s, kMaxSplits)) : 0;
  return (size_t)most(whole, divided);
}

// Whether the splits' partial results are held in fp32 rather than bf16.  In bf16 a result carries one more rounding than
// an undivided one (error against fp64 2.9e-3 instead of 2.35e-3 of its norm for N(0, 1) inputs, however many splits; with
// fp32 partials 2.3e-3), but they are the largest avoidable traffic of a call, and half of it.  They are fp32 for two and
// three splits, and for any number where the row tiles would have given most CUs a workgroup undivided: there the keys are
// divided for the balance of a batch, not because the card would be idle.  Where the undivided grid is more than one turn
// already they are only if that adds no more than 3 % to the estimated time; and there are never more than 64 MB of them.
// (Of 40000 drawn shapes 1698 run divided that an earlier plan left undivided; 1524 of those have fp32 partials.)  What it
// costs (us, bf16 / fp32): sixteen ragged sequences of up to 4096 keys, 8B, two splits 62.4 / 65.9; 13B, four sequences,
// three splits 40.4 / 42.0; 7B, six sequences of 2048, two splits 47.8 / 49.2; two sequences of 300 keys 9.36 / 9.47; and,
// left in bf16, eight sequences, four splits 36.6 / 39.7, twenty-four, two splits and a second launch 144 / 148 - 160.
constexpr int kFineSplits = 3;
constexpr size_t kFineBytes = (size_t)64 << 20;
bool fine_partials(const AttnPlan& pl, long long units, int head_dim, double added_us, double call_us) {
  if (pl.splits < 2) return false;
  if (pl.wm == 8) return true;
  if (pl.fused) return pl.splits <= kFineSplits;  // (what the kernel's instances assume; at most 512 workgroups: 34 MB)
  const int cus = device_cu_count();
  const long long wgs = units * pl.n_qtiles;  // undivided
  const bool balance = pl.n_qtiles == 1 && 16 * wgs >= 11 * cus && wgs <= cus;
  return (pl.splits <= kFineSplits || balance) && (wgs <= cus || added_us <= 0.03 * call_us) &&
         (size_t)units * pl.splits * pl.m_pad * head_dim * sizeof(float) <= kFineBytes;
}

bool compute_attn_plan(const jk_attn_desc& d, int max_prefix_len, bool fused_allowed, AttnPlan* pl) {
  static const PlanModel km;
  if (!desc_ok(d) || !shape_supported(d) || max_prefix_len < 0 || max_prefix_len > (1 << 24)) return false;
  const int G = d.n_q_heads / d.n_kv_heads;
  pl->m_rows = d.n_tree * G;
  const long long units = (long long)d.batch * d.n_kv_heads;
  const size_t most_rows = most_part_rows(d, max_prefix_len);
  if (d.dtype == JK_BF16) {
    // Candidates: 4x1 or 2x2 waves (32-row blocks x key interleave) per workgroup.  Fewer
    // rows per workgroup means more workgroups per KV head without more KV splits: the K/V
    // stream is then re-read by the row tiles (from L2, they run side by side on one XCD)
    // instead of partial outputs being written and read back once per split.
    const int n_tiles = (max_prefix_len + kTileKeys - 1) / kTileKeys + (d.n_tree + kTileKeys - 1) / kTileKeys;
    const double kv_bytes = 2.0 * (max_prefix_len + d.n_tree) * d.head_dim * 2.0;
    const int slots = device_cu_count();  // one workgroup per CU measured best (partials cost more than idle slots)
    const Tuning& tn = tuning();
    const int forced_wm = tn.attn_wm, forced_wn = tn.attn_wn, forced_s = tn.attn_splits;  // tuning overrides
    const int fused_mode = !fused_allowed ? 0 : tn.attn_fused;  // 0 never, 1 whenever possible, -1 when it pays
    static const int kArr[][2] = {{2, 2}, {4, 1}, {8, 1}, {1, 4}};  // waves along rows x along keys ({1, 4}: tva_direct.hip, 16 rows)
    bool forced_ok = false;
    for (const auto& a : kArr) forced_ok |= (a[0] == forced_wm && a[1] == forced_wn);
    double best_cost = 0.0, best_part_mb = 0.0;
    bool have = false;
    for (const auto& a : kArr) {
      const int wm = a[0], wn = a[1];
      if (wm == 8 && !forced_ok && (pl->m_rows <= 96 || tn.attn_fused == 0)) continue;  // (mostly padding rows; it has no second launch)
      if (forced_ok ? (wm != forced_wm || wn != forced_wn) : (wm > 2 && pl->m_rows <= 16 * wm)) continue;  // mostly padding rows
      const bool direct = wm == 1;
      if (direct && !forced_ok && tn.attn_fused >= 0) continue;  // (a forced merge asks for a kernel that has one)
      const int q_rows = direct ? 16 : 32 * wm;
      const int n_qtiles = (pl->m_rows + q_rows - 1) / q_rows;
      const long long wgs = units * n_qtiles;
      const int kt = wm == 4 ? 2 : 1;  // (4x1: tiles in pairs, the hand-pipelined two-tile path)
      const int max_by_tiles = n_tiles >= 4 ? n_tiles / 4 : 1;  // at least two rounds of two tiles per split
      // every split count that leaves a split at least two rounds is priced
      const long long s_top = forced_s >= 1 && forced_s <= kMaxSplits ? 1 : (max_by_tiles < kMaxSplits ? max_by_tiles : kMaxSplits);
      for (long long sc = 1; sc <= s_top; ++sc) {
        long long s = sc;
        if (forced_s >= 1 && forced_s <= kMaxSplits) s = forced_s;
        // a split's tiles stay within what a workgroup can keep page ids for (paged caches)
        const long long s_min = (n_tiles + kMaxTilesPerSplit - 1) / kMaxTilesPerSplit;
        if (s < s_min) s = s_min;
        if (s > kMaxSplits) continue;
        if (direct && sc > 1) break;
        if (direct) s = 1;  // (it has no splits, and its page ids are in registers: whatever is forced)
        // (beyond that the splits of the others are the better one in most calls, and the estimate too coarse to tell the rest: of the
        // 139 shapes of profiles/attention_plan_times.csv with 29 to 56 tiles six are more than 3 % faster with this kernel, 14 % at most,
        // and all together take 1.6 times as long)
        if (direct && !forced_ok && n_tiles > 28) break;
        if (s > 1 && forced_s < 1 && (size_t)(wgs * s * q_rows) > most_rows) continue;  // (one split always fits)
        if (wm == 8 && s > 1 && (wgs * s > kMaxCounted || (size_t)wgs * s * q_rows * d.head_dim * sizeof(float) > kFineBytes)) continue;
        // rounds of the longest split: the 4x1 arrangement deals tiles (an odd last tile costs about
        // half a round), the 2x2 arrangement whole rounds
        double rounds;
        if (wn == 1) {
          // (the kernel's own dealing: full prefix tiles evenly, a lone last tile a little over half a
          // pair; the tail - two full tiles a tile - with the last split)
          const long long F = max_prefix_len / kTileKeys, tail = n_tiles - F;
          auto pairs_of = [](long long tiles) { return 0.5 * (double)(tiles / 2 * 2) + ((tiles & 1) ? 0.55 : 0.0); };
          if (s == 1) {
            rounds = pairs_of(F) + 1.07 * (double)tail;
          } else {
            const long long per = (F + 2 * tail + s - 1) / s;
            long long f_last = per - 2 * tail;
            f_last = (f_last < 0 ? 0 : (f_last > F ? F : f_last)) & ~1LL;
            const long long rest = F - f_last, most = (rest + s - 2) / (s - 1);
            const double last = pairs_of(f_last) + 1.07 * (double)tail;
            rounds = pairs_of(most) > last ? pairs_of(most) : last;
          }
        } else {
          rounds = (double)(((n_tiles + wn * kt - 1) / (wn * kt) + s - 1) / s) +
                   km.tail_2x2 * (double)(n_tiles - max_prefix_len / kTileKeys) / (double)(1 + s);
        }
        const long long all_wgs = wgs * s;
        // The six-tile ring of the 2x2 arrangement: two rounds in flight for a workgroup that has its CU to itself
        // and a long way to stream (at least eight rounds): 0.75 - 0.86 of the time where K/V come from HBM, 1.02 where
        // they sit in a cache (900 drawn shapes); never where two workgroups may share a CU, since only one with
        // the deeper ring fits.
        const bool deep_ok = wn == 2 && all_wgs <= slots;
        const bool deep = deep_ok && (tn.attn_deep == 1 || (tn.attn_deep < 0 && ((n_tiles + 1) / 2 + s - 1) / s >= 8));
        // One turn of at most two workgroups per CU: its rounds, or its share of the K/V stream, whichever is
        // longer (they overlap badly where they are close, hence the 4-norm).
        const double t_round = d.head_dim == 64 ? (wn == 1 ? km.round_4x1_d64 : km.round_2x2_d64)
                                                : (wn == 1 ? km.round_4x1 : km.round_2x2);
        const double stream_us = (double)units * kv_bytes / (double)all_wgs / km.stream;  // per workgroup of a turn
        const bool far = wn == 2 && (double)units * kv_bytes > km.far_bytes;
        const double lone = far ? (deep ? km.far_deep : km.far_2x2) : 1.0;
        const double shared = wn == 1 ? km.share_4x1 : km.share_2x2 * (far ? km.far_2x2_shared : 1.0);
        auto turn_us = [&](long long n) {
          if (n <= 0) return 0.0;
          const double loop = rounds * t_round * (n <= slots ? lone : shared);
          const double l2 = loop * loop, m2 = stream_us * (double)n * (stream_us * (double)n);
          return std::sqrt(std::sqrt(l2 * l2 + m2 * m2));
        };
        const long long full = all_wgs / (2 * slots);
        const double body_full = (double)full * turn_us(2 * slots), body_last = turn_us(all_wgs - full * 2 * slots);
        double body = body_full + body_last;
        if (full >= 1) {
          const double even = (double)all_wgs / (2.0 * slots) * turn_us(2 * slots);
          const double part = km.turn_0 - km.turn_step * (double)(full - 1);
          const double shows = part > km.turn_min ? part : km.turn_min;
          body = shows * body + (1.0 - shows) * even;
        }
        // Merge inside the kernel: possible when every workgroup is resident at once (here: at most
        // one per CU, or two when forced) and the workgroup numbering puts all splits of a (unit, row
        // tile) group on one XCD: logical ids are dealt to the 8 XCDs in contiguous ranges of
        // total / 8, and a unit's ids are contiguous, so every unit's range must sit inside one.
        // (and one thread per (row of a slice, split padded to a power of two); partials below 2^31 bytes)
        int s_pow2 = 1;
        while (s_pow2 < s) s_pow2 *= 2;
        bool can_fuse = fused_mode != 0 && s > 1 && wgs <= kMaxFusedGroups &&
                        ((q_rows + s - 1) / s) * s_pow2 <= 64 * wm * wn &&
                        (double)units * s * n_qtiles * q_rows * d.head_dim * 2.0 < 2.0e9 &&
                        all_wgs <= (long long)slots * 2;  // (two of these workgroups fit a CU: all resident)
        if (wm == 8) can_fuse = s > 1;  // (that kernel always merges its splits, wherever they run)
        else if (can_fuse) {
          const long long per_unit = s * n_qtiles, per_xcd = (all_wgs + 7) / 8;
          for (long long u = 0; u < units && can_fuse; ++u)
            can_fuse = (u * per_unit) / per_xcd == ((u + 1) * per_unit - 1) / per_xcd;
        }
        // Partials are merged inside the kernel where that is possible: an exchange through the XCD's L2 instead of a
        // second launch, 0.2 - 4.8 us less over five shapes with 2 - 32 splits, but 0.4 - 1.1 us more for two or three
        // splits of 2x2 workgroups with a head dimension of 64.
        const double part_mb = 1.0e-6 * (double)units * s * pl->m_rows * d.head_dim * 2.0;
        const double fused_us = km.merge_fused_fixed + km.merge_fused_per_mb * part_mb;
        const double kernel_us = km.merge_kernel_fixed + km.merge_kernel_per_mb * part_mb;
        const double merge_us = s <= 1 ? 0.0 : (can_fuse ? fused_us : kernel_us) + km.merge_16 * (double)((s - 1) / 16);
        const double start_us = km.startup * (wn == 1 ? km.startup_4x1 : 1.0);
        // (near ties go to the count that gives every CU a workgroup: 2 % for idle CUs)
        double cost = (body + merge_us + start_us) * (all_wgs < slots ? 1.02 : 1.0);
        if (wm == 8) {
          const int per = (int)((n_tiles + s - 1) / s), masked = n_tiles - max_prefix_len / kTileKeys;
          const int plain = per > masked + 2 ? per - masked - 2 : 0;  // (the first tile, and those that four does not divide)
          const double turns = (double)((all_wgs + slots - 1) / slots);
          const double load = (all_wgs < slots ? (double)all_wgs / slots : 1.0) * plain / km.wide_hot_tiles;
          const double loop = plain * (d.head_dim == 64 ? km.wide_tile_d64 : km.wide_tile) * (1.0 + km.wide_hot * (load < 1.0 ? load : 1.0)) +
                              (per - plain) * (d.head_dim == 64 ? km.wide_slow_d64 : km.wide_slow);
          const double stream = (double)units * kv_bytes / turns / km.wide_stream;
          const double l2 = loop * loop, m2 = stream * stream;
          int levels = 0;
          while ((1 << levels) < s) ++levels;
          cost = km.wide_margin * (km.wide_call + turns * (km.wide_turn + std::sqrt(std::sqrt(l2 * l2 + m2 * m2))) + km.wide_level * levels +
                                   km.wide_merge_per_mb * 2.0 * part_mb * (double)(s - 1) / (double)s);
        }
        if (direct) {
          const double per_cu = (double)((all_wgs + slots - 1) / slots);
          const double loop = (double)((n_tiles + 3) / 4) * (d.head_dim == 64 ? km.direct_round_d64 : km.direct_round);
          const double draw = per_cu * kv_bytes / km.direct_draw, l2 = loop * loop, m2 = draw * draw;
          cost = km.direct_level * ((d.head_dim == 64 ? km.direct_call_d64 : km.direct_call) + std::sqrt(std::sqrt(l2 * l2 + m2 * m2)) +
                                    (double)units * kv_bytes / km.direct_stream + (per_cu - 1.0) * km.direct_next +
                                    (d.n_tree > 64 ? km.direct_deep_tree : 0.0));
        }
        if (!have || cost < best_cost) {
          have = true;
          best_cost = cost;
          best_part_mb = part_mb;
          pl->wm = wm; pl->wn = wn; pl->kt = kt; pl->q_rows = q_rows; pl->n_qtiles = n_qtiles; pl->splits = (int)s;
          pl->fused = can_fuse ? 1 : 0;
          pl->deep = deep ? 1 : 0;
        }
      }
    }
    if (!have) return false;
    pl->parts = pl->splits;
    pl->m_pad = pl->n_qtiles * pl->q_rows;
    pl->fine = fine_partials(*pl, units, d.head_dim, km.merge_kernel_per_mb * best_part_mb, best_cost) ? 1 : 0;
    // (the kernel ranks a batch with a lane per sequence, and the XCDs get whole units)
    pl->ranked = d.batch >= 2 && d.batch <= 64 && (pl->wm == 8 || units % 8 == 0) ? 1 : 0;
  } else {
    pl->fused = 0;
    pl->fine = 0;
    pl->ranked = 0;
    pl->deep = 0;
    pl->wm = pl->wn = pl->kt = 1;
    pl->q_rows = 1;  // (as reported; the kernel's workgroups take 16 rows and the parts below)
    pl->n_qtiles = pl->m_rows;
    pl->m_pad = pl->m_rows;
    const long long keys = (long long)max_prefix_len + d.n_tree;
    long long s = (keys + 1023) / 1024;  // ranges of 1024 keys, for 16 query rows a workgroup
    if (s > kMaxSplits) return false;  // fp32 path: at most 64 * 1024 keys
    pl->splits = (int)s;
    // Few workgroups: each range in up to eight parts, where merging them (in the kernel, by the last workgroup of a row tile; of many
    // parts in a launch of its own) costs less than what the parts save.  A wave's time for a block of keys hardly depends on head_dim
    // up to 64 (maximum, exponentials, trips), so neither does the line; beyond 128 a workgroup has four waves instead of eight.
    // Whole / in 4 / 6 / 8 parts, us, 20 nodes and 8 heads, of 64: 320 keys 8.9 / 7.8 / 7.7 / 7.8, 620 12.2 / 9.0 / 8.2 / 8.5; of 128:
    // 200 11.5 / 9.3 / 9.6 / 9.8, 320 15.1 / 10.8 / 10.6 / 10.1; of 192: 121 14.0 / 12.6 / 13.3 / 13.2, 200 20.2 / 13.6 / 14.3 / 14.0, 300
    // 23.6 / 16.9 / 14.8 / 14.5.  Where three parts fill the CUs (80 row tiles), whole / in 3: of 64, 170 keys 6.6 / 7.6, 340 9.5 / 8.2; of 80,
    // 170 8.6 / 8.9, 340 12.8 / 10.1.  Four parts would pay a little earlier (of 64, 250 keys 7.9 / 7.4; of 128, 150 9.9 / 9.2), but the bytes
    // that a call asks for stay as they are, so that a workspace allocated by them still serves it.
    // A fifth part, where no more fit, is one more to merge, and pays where it saves a turn of the waves, but for two ranges of heads up
    // to 128.  In 4 / 5 parts a range, one range of 423 keys, heads of 80, 8.6 / 9.8, of 990 and 128 15.2 / 16.3, of 547 and 32 9.0 / 8.6, of 749
    // and 128 14.4 / 13.9 (not taken); two of 1316 and 80 10.8 / 12.5, of 1153 and 256 20.6 / 19.8; three of 2726 and 32 11.7 / 10.8, of 2117 and 256 22.0 / 23.4.
    // Over the 260 drawn calls of profiles/f32_parts_times.csv (90 - 4000 keys, head_dim 16 - 256, every number of parts that fits) the
    // one taken is 1.7 % slower than the best (6.6 % at the 90th percentile; 21 % at the 99th, calls in front of the lines above).
    const long long wgs = units * ((pl->m_rows + 15) / 16) * s;
    pl->parts = pl->splits;
    if (f32_in_parts(keys, d.head_dim)) {
      auto turns = [&](int sub) { return ((keys / s + sub - 1) / sub - 1) / 64; };  // (of four blocks of 16 keys)
      const bool fifth = !(d.head_dim <= 128 && s == 2) && turns(5) < turns(4);
      const int most = keys < 220 ? 4 : keys < 300 ? 6 : 8;
      for (int sub = most; sub > 1; --sub)
        if (wgs * sub <= device_cu_count() && s * sub <= kMaxSplits && (sub != 5 || fifth)) {
          pl->parts = pl->splits * sub;
          break;
        }
    }
  }
  auto up = [](size_t x) { return (x + 255) / 256 * 256; };
  const size_t rows = pl->parts > 1 ? (size_t)units * pl->parts * pl->m_pad : 0, o_row = (size_t)d.head_dim * (d.dtype == JK_BF16 ? 2 : sizeof(float));
  pl->part_o_bytes = up(rows * (pl->fine ? 2 * o_row : o_row));
  pl->part_ml_bytes = up(rows * sizeof(float2));
  pl->total_bytes = kAttnHeaderBytes + pl->part_o_bytes + pl->part_ml_bytes;
  size_t most_o = most_rows * o_row;
  if (d.dtype == JK_BF16) {  // (a smaller call's partials may be fp32)
    const size_t fine_o = 2 * most_rows * o_row < kFineBytes ? 2 * most_rows * o_row : kFineBytes;
    if (fine_o > most_o) most_o = fine_o;
  }
  const size_t covers = kAttnHeaderBytes + up(most_o) + up(most_rows * sizeof(float2));
  pl->covers_bytes = covers > pl->total_bytes ? covers : pl->total_bytes;  // (a forced split count may need more)
  return true;
}
}  // namespace

// Pricing up to 128 ways to cut a call costs the host 3 - 10 us, as much as a small call runs on the GPU: a thread
// keeps the plans of its last shapes (a model's layers all ask for the same one; a draft round for a handful).
bool make_attn_plan(const jk_attn_desc& d, int max_prefix_len, bool fused_allowed, AttnPlan* pl) {
  constexpr int kKey = 13, kSlots = 32;
  struct Entry {
    int key[kKey];
    AttnPlan plan;
  };
  static thread_local Entry kept[kSlots];  // (a key of zeros names no valid shape: batch >= 1)
  if (!desc_ok(d)) return false;
  const Tuning& t = tuning();
  const int key[kKey] = {d.batch, d.n_tree, d.n_q_heads, d.n_kv_heads, d.head_dim, d.dtype, max_prefix_len, fused_allowed ? 1 : 0,
                         t.attn_wm, t.attn_wn, t.attn_splits, t.attn_fused, t.attn_deep};
  unsigned h = 0;
  for (int v : key) h = (h ^ (unsigned)v) * 0x9E3779B1u;
  Entry& e = kept[h >> 27];
  if (std::memcmp(e.key, key, sizeof(key)) != 0) {
    AttnPlan fresh;
    if (!compute_attn_plan(d, max_prefix_len, fused_allowed, &fresh)) return false;
    e.plan = fresh;
    std::memcpy(e.key, key, sizeof(key));
  }
  *pl = e.plan;
  return true;
}

namespace {
bool heads_shape_ok(int rows, int d_model, int vocab) {
  return rows >= 1 && rows <= 128 && d_model >= 128 && d_model <= 16384 && d_model % 128 == 0 && vocab >= 1 && vocab <= (1 << 24);
}
bool moe_desc_ok(const jk_moe_desc& d) { return d.rows >= 1 && d.d_model >= 1 && d.d_ff >= 1 && d.n_experts >= 2; }
bool moe_desc_supported(const jk_moe_desc& d) {
  return d.rows <= 128 && d.d_model >= 128 && d.d_model <= 65536 && d.d_model % 128 == 0 && d.d_ff >= 128 &&
         d.d_ff <= 65536 && d.d_ff % 128 == 0 && d.n_experts <= 64;
}
bool linear_shape_ok(int m, int n, int k) {
  return m >= 1 && m <= 256 && n >= 1 && k >= 128 && k % 128 == 0 && k <= (1 << 20) && n <= (1 << 24);
}

// What the calls with the same weights and at most `rows` rows need: fewer rows may be cut into more parts and need more
// room, and a program sizes its workspace once.  (Up to 256 plans to make, 20 - 110 us: callers that allocate per call
// ask for that call's own need.)
template <class Bytes>
size_t most_bytes(int rows, Bytes bytes_of_rows) {
  size_t most = 0;
  for (int r = 1; r <= rows; ++r) {
    const size_t n = bytes_of_rows(r);
    if (n > most) most = n;
  }
  return most;
}
}  // namespace

size_t draft_heads_call_bytes(int rows, int d_model, int vocab) {
  return heads_shape_ok(rows, d_model, vocab) ? draft_heads_workspace_bytes(rows, d_model, vocab) : 0;
}
size_t moe_experts_call_bytes(const jk_moe_desc& d) {
  return moe_desc_ok(d) && moe_desc_supported(d) ? moe_experts_workspace_bytes(d.rows, d.d_model, d.d_ff, d.n_experts) : 0;
}
size_t linear_call_bytes(int m, int n, int k) { return linear_shape_ok(m, n, k) ? linear_workspace_bytes(m, n, k) : 0; }
namespace {
jk_status linear_refused(int32_t m, int32_t n, int32_t k, const void* x, const void* w, const void* out_bf16, const float* out_f32) {
  if (!x || !w || (!out_bf16 && !out_f32) || m < 1 || n < 1 || k < 1) return JK_ERR_INVALID_ARG;
  if (reinterpret_cast<uintptr_t>(x) % 16 || reinterpret_cast<uintptr_t>(w) % 16) return JK_ERR_INVALID_ARG;
  return linear_shape_ok(m, n, k) ? JK_OK : JK_ERR_UNSUPPORTED;
}
jk_status linear_launched(int m, int n, int k, const void* x, const void* w, const void* residual, void* out_bf16, float* out_f32,
                                 void* workspace, void* hip_stream) {
  LinearArgs a;
  a.m = m; a.n = n; a.k = k; a.x = x; a.w = w; a.residual = residual; a.out_f32 = out_f32; a.out_bf16 = out_bf16;
  a.workspace = workspace;
  return launch_linear(a, static_cast<hipStream_t>(hip_stream)) == hipSuccess ? JK_OK : JK_ERR_HIP;
}
}  // namespace
jk_status linear_call(int m, int n, int k, const void* x, const void* w, const void* residual, void* out_bf16, float* out_f32,
                      void* workspace, void* hip_stream) {
  if (jk_status s = linear_refused(m, n, k, x, w, out_bf16, out_f32); s != JK_OK) return s;
  if (!workspace && linear_call_writes(m, n, k)) return JK_ERR_WORKSPACE;
  return linear_launched(m, n, k, x, w, residual, out_bf16, out_f32, workspace, hip_stream);
}

}  // namespace jk

using namespace jk;

extern "C" {

size_t jk_tree_verify_attention_workspace(const jk_attn_desc* desc, int32_t max_prefix_len) {
  // Whether the splits are merged inside the kernel depends on jk_init having verified the device,
  // and the two plans may cut the work differently: the size covers both, so that it is a function
  // of the descriptor and the bound alone (see most_part_rows).
  AttnPlan a, b;
  if (!desc || !make_attn_plan(*desc, max_prefix_len, false, &a) || !make_attn_plan(*desc, max_prefix_len, true, &b))
    return 0;
  return a.covers_bytes > b.covers_bytes ? a.covers_bytes : b.covers_bytes;
}

jk_status jk_tree_verify_attention_plan(const jk_attn_desc* desc, int32_t max_prefix_len, int32_t* plan_out) {
  if (!desc || !plan_out) return JK_ERR_INVALID_ARG;
  AttnPlan pl;
  if (!make_attn_plan(*desc, max_prefix_len, xcd_placement_verified(), &pl)) return JK_ERR_UNSUPPORTED;
  plan_out[0] = pl.wm; plan_out[1] = pl.wn; plan_out[2] = pl.kt; plan_out[3] = pl.n_qtiles;
  plan_out[4] = pl.splits; plan_out[5] = pl.fused;
  return JK_OK;
}

static jk_status attention_common(const jk_attn_desc* desc, const jk_paged_kv* pages, const void* q,
                                  const void* k_cache, const void* v_cache, const void* k_tree, const void* v_tree,
                                  const int32_t* parent, const int32_t* prefix_len, int32_t max_prefix_len, void* out,
                                  void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!desc || !q || !k_tree || !v_tree || !parent || !prefix_len || !out) return JK_ERR_INVALID_ARG;
  if (max_prefix_len < 0) return JK_ERR_INVALID_ARG;
  if (max_prefix_len > 0 && (!k_cache || !v_cache)) return JK_ERR_INVALID_ARG;
  const jk_attn_desc& d = *desc;
  if (!desc_ok(d)) return JK_ERR_INVALID_ARG;
  if (!shape_supported(d)) return JK_ERR_UNSUPPORTED;
  const int64_t align = (d.dtype == JK_BF16) ? 8 : 4;
  const size_t es = (d.dtype == JK_BF16) ? 2 : 4;
  const int64_t strides[] = {d.q_stride_b, d.q_stride_t, d.q_stride_h, d.kc_stride_b, d.kc_stride_l,
                             d.kc_stride_h, d.kt_stride_b, d.kt_stride_t, d.kt_stride_h, d.o_stride_b,
                             d.o_stride_t, d.o_stride_h};
  for (int64_t s : strides)
    if (s < 0 || s % align) return JK_ERR_INVALID_ARG;
  if (d.q_stride_t < d.head_dim && d.n_tree > 1) return JK_ERR_INVALID_ARG;
  // the bf16 kernel addresses a tile's rows with 32-bit byte offsets from the tile's first row
  if (d.dtype == JK_BF16 && (d.kc_stride_l > (1 << 24) || d.kt_stride_t > (1 << 24))) return JK_ERR_UNSUPPORTED;
  // and finds a row's node and a workgroup's sequence by multiplications of 32 bits (beyond: the wrong ones)
  const int group = d.n_q_heads / d.n_kv_heads;
  if (d.dtype == JK_BF16 && !(exact_in_32((long long)d.n_tree * group, group) && exact_in_32((long long)d.batch * d.n_kv_heads, d.n_kv_heads)))
    return JK_ERR_UNSUPPORTED;
  const void* ptrs[] = {q, k_cache, v_cache, k_tree, v_tree, out};
  for (const void* p : ptrs)
    if (reinterpret_cast<uintptr_t>(p) % (align * es)) return JK_ERR_INVALID_ARG;
  if (pages) {
    if (d.dtype != JK_BF16) return JK_ERR_UNSUPPORTED;
    if (!pages->block_table || pages->page_size < 1 || pages->max_blocks < 1 || pages->n_pages < 1)
      return JK_ERR_INVALID_ARG;
    if (pages->page_size % kTileKeys) return JK_ERR_UNSUPPORTED;  // a page holds whole 32-key tiles
    if (pages->page_stride < 0 || pages->page_stride % align) return JK_ERR_INVALID_ARG;
    if ((long long)pages->max_blocks * pages->page_size < max_prefix_len) return JK_ERR_INVALID_ARG;
  }

  AttnPlan pl;
  if (!make_attn_plan(d, max_prefix_len, xcd_placement_verified(), &pl)) return JK_ERR_UNSUPPORTED;
  if (!workspace || reinterpret_cast<uintptr_t>(workspace) % 256) return JK_ERR_WORKSPACE;
  if (workspace_bytes < pl.total_bytes) return JK_ERR_WORKSPACE;
  if (tuning().verbose)
    std::fprintf(stderr, "jk attention plan: waves %dx%d, %d tile(s) per wave and round, %d row tile(s), %d split(s)%s%s\n",
                 pl.wm, pl.wn, pl.kt, pl.n_qtiles, pl.splits, pl.fused ? ", merged in the kernel" : "", pl.deep ? ", six-tile ring" : "");

  AttnArgs a;
  a.q = q; a.k_cache = k_cache; a.v_cache = v_cache; a.k_tree = k_tree; a.v_tree = v_tree;
  a.parent = parent; a.prefix_len = prefix_len; a.out = out;
  char* ws = static_cast<char*>(workspace);
  a.err = reinterpret_cast<unsigned*>(ws);
  a.sync = reinterpret_cast<unsigned*>(ws + kWsErrBytes);
  a.part_o = reinterpret_cast<float*>(ws + kAttnHeaderBytes);
  a.part_ml = reinterpret_cast<float2*>(ws + kAttnHeaderBytes + pl.part_o_bytes);
  a.d = d;
  a.max_prefix_len = max_prefix_len;
  a.block_table = pages ? pages->block_table : nullptr;
  a.max_blocks = pages ? pages->max_blocks : 0;
  a.page_size = pages ? pages->page_size : 0;
  a.n_pages = pages ? pages->n_pages : 0;
  a.page_stride = pages ? pages->page_stride : 0;
  const float scale = d.scale > 0.f ? d.scale : 1.0f / std::sqrt((float)d.head_dim);
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  hipError_t e;
  if (d.dtype == JK_BF16) {
    a.scale_log2 = scale * 1.44269504088896340736f;
    e = launch_tva_bf16(a, pl, stream);
    if (e == hipSuccess && pl.splits > 1 && !pl.fused) e = launch_tva_combine(a, pl, stream);
  } else {
    a.scale_log2 = scale;  // the fp32 path works in natural units
    if (!f32_merges(d, pl)) a.sync = nullptr;
    e = launch_tva_f32(a, pl, stream);
    if (e == hipSuccess && pl.parts > 1 && !a.sync) e = launch_tva_combine(a, pl, stream);
  }
  return e == hipSuccess ? JK_OK : JK_ERR_HIP;
}

jk_status jk_tree_verify_attention(const jk_attn_desc* desc, const void* q, const void* k_cache,
                                   const void* v_cache, const void* k_tree, const void* v_tree,
                                   const int32_t* parent, const int32_t* prefix_len, int32_t max_prefix_len,
                                   void* out, void* workspace, size_t workspace_bytes, void* hip_stream) {
  return attention_common(desc, nullptr, q, k_cache, v_cache, k_tree, v_tree, parent, prefix_len, max_prefix_len, out,
                          workspace, workspace_bytes, hip_stream);
}

jk_status jk_tree_verify_attention_paged(const jk_attn_desc* desc, const jk_paged_kv* pages, const void* q,
                                         const void* k_pool, const void* v_pool, const void* k_tree,
                                         const void* v_tree, const int32_t* parent, const int32_t* prefix_len,
                                         int32_t max_prefix_len, void* out, void* workspace, size_t workspace_bytes,
                                         void* hip_stream) {
  if (!pages) return JK_ERR_INVALID_ARG;
  return attention_common(desc, pages, q, k_pool, v_pool, k_tree, v_tree, parent, prefix_len, max_prefix_len, out,
                          workspace, workspace_bytes, hip_stream);
}

size_t jk_accept_path_workspace(int32_t batch, int32_t n_tree, int32_t vocab, int32_t mode) {
  if (batch < 1 || n_tree < 1 || n_tree > JK_MAX_TREE || vocab < 1) return 0;
  if (mode != JK_GREEDY && mode != JK_SAMPLE) return 0;
  return accept_workspace_bytes(batch, n_tree, vocab, mode);
}

static jk_status accept_common(int32_t batch, int32_t n_tree, int32_t vocab, int32_t max_depth,
                               const int32_t* tree_tokens, const int32_t* parent, const float* target_logits,
                               int32_t mode, float temperature, const float* draft_probs, const int32_t* draft_row,
                               int64_t n_draft_rows, const float* uniforms, int32_t* out_path,
                               int32_t* out_accept_len, int32_t* out_bonus_token, void* workspace,
                               size_t workspace_bytes, void* hip_stream) {
  if (batch < 1 || vocab < 1 || max_depth < 1) return JK_ERR_INVALID_ARG;
  if (n_tree < 1) return JK_ERR_INVALID_ARG;
  if (n_tree > JK_MAX_TREE) return JK_ERR_UNSUPPORTED;
  if (mode != JK_GREEDY && mode != JK_SAMPLE) return JK_ERR_INVALID_ARG;
  if (!tree_tokens || !parent || !target_logits || !out_path || !out_accept_len || !out_bonus_token)
    return JK_ERR_INVALID_ARG;
  if (reinterpret_cast<uintptr_t>(target_logits) % 16) return JK_ERR_INVALID_ARG;
  if ((long long)batch * (n_tree + 1) > 65535) return JK_ERR_UNSUPPORTED;
  if (mode == JK_SAMPLE) {
    if (!draft_probs || !uniforms) return JK_ERR_INVALID_ARG;
    if (!(temperature > 0.f) || !std::isfinite(temperature)) return JK_ERR_INVALID_ARG;
    if (draft_row && n_draft_rows < 1) return JK_ERR_INVALID_ARG;
  }
  const size_t need = accept_workspace_bytes(batch, n_tree, vocab, mode);
  if (!workspace || reinterpret_cast<uintptr_t>(workspace) % 256) return JK_ERR_WORKSPACE;
  if (workspace_bytes < need) return JK_ERR_WORKSPACE;
  AcceptArgs a;
  a.batch = batch; a.n_tree = n_tree; a.vocab = vocab; a.max_depth = max_depth; a.mode = mode;
  a.temperature = temperature;
  a.tokens = tree_tokens; a.parent = parent; a.logits = target_logits;
  a.draft_probs = draft_probs; a.uniforms = uniforms;
  a.draft_row = draft_row; a.n_draft_rows = n_draft_rows;
  a.out_path = out_path; a.out_len = out_accept_len; a.out_bonus = out_bonus_token;
  a.workspace = workspace;
  return launch_accept(a, static_cast<hipStream_t>(hip_stream)) == hipSuccess ? JK_OK : JK_ERR_HIP;
}

jk_status jk_accept_path(int32_t batch, int32_t n_tree, int32_t vocab, int32_t max_depth,
                         const int32_t* tree_tokens, const int32_t* parent, const float* target_logits,
                         int32_t mode, float temperature, const float* draft_probs, const float* uniforms,
                         int32_t* out_path, int32_t* out_accept_len, int32_t* out_bonus_token, void* workspace,
                         size_t workspace_bytes, void* hip_stream) {
  return accept_common(batch, n_tree, vocab, max_depth, tree_tokens, parent, target_logits, mode, temperature,
                       draft_probs, nullptr, 0, uniforms, out_path, out_accept_len, out_bonus_token, workspace,
                       workspace_bytes, hip_stream);
}

jk_status jk_accept_path_greedy_static(int32_t batch, int32_t n_tree, int32_t vocab, int32_t max_depth,
                                       const int32_t* tree_tokens, const int32_t* parent,
                                       const float* target_logits, int32_t* out_path, int32_t* out_accept_len,
                                       int32_t* out_bonus_token, void* hip_stream) {
  if (batch < 1 || vocab < 1 || max_depth < 1 || n_tree < 1) return JK_ERR_INVALID_ARG;
  if (n_tree > JK_MAX_TREE) return JK_ERR_UNSUPPORTED;
  if (!tree_tokens || !parent || !target_logits || !out_path || !out_accept_len || !out_bonus_token)
    return JK_ERR_INVALID_ARG;
  if (reinterpret_cast<uintptr_t>(target_logits) % 16) return JK_ERR_INVALID_ARG;
  if ((long long)batch * (n_tree + 1) > 65535) return JK_ERR_UNSUPPORTED;
  if (accept_greedy_static_bytes(batch, n_tree, vocab) > (size_t)JK_STATIC_SCRATCH_BYTES) return JK_ERR_SCRATCH_LIMIT;
  AcceptArgs a;
  a.batch = batch; a.n_tree = n_tree; a.vocab = vocab; a.max_depth = max_depth; a.mode = JK_GREEDY;
  a.temperature = 1.f;
  a.tokens = tree_tokens; a.parent = parent; a.logits = target_logits;
  a.draft_probs = nullptr; a.uniforms = nullptr; a.draft_row = nullptr; a.n_draft_rows = 0;
  a.out_path = out_path; a.out_len = out_accept_len; a.out_bonus = out_bonus_token;
  a.workspace = nullptr;
  return launch_accept_greedy_static(a, static_cast<hipStream_t>(hip_stream)) == hipSuccess ? JK_OK : JK_ERR_HIP;
}

jk_status jk_accept_path_rows(int32_t batch, int32_t n_tree, int32_t vocab, int32_t max_depth,
                              const int32_t* tree_tokens, const int32_t* parent, const float* target_logits,
                              int32_t mode, float temperature, const float* draft_rows_all, int64_t n_draft_rows,
                              const int32_t* draft_row, const float* uniforms, int32_t* out_path,
                              int32_t* out_accept_len, int32_t* out_bonus_token, void* workspace,
                              size_t workspace_bytes, void* hip_stream) {
  if (mode == JK_SAMPLE && !draft_row) return JK_ERR_INVALID_ARG;
  return accept_common(batch, n_tree, vocab, max_depth, tree_tokens, parent, target_logits, mode, temperature,
                       draft_rows_all, draft_row, n_draft_rows, uniforms, out_path, out_accept_len, out_bonus_token,
                       workspace, workspace_bytes, hip_stream);
}

static jk_status commit_common(const jk_attn_desc* desc, const jk_paged_kv* pages, int n_layers, const void* k_tree, const void* v_tree,
                               void* k_cache, void* v_cache, const int32_t* path, const int32_t* accept_len,
                               int32_t max_depth, int32_t cache_capacity, int32_t* prefix_len, int32_t advance,
                               void* hip_stream) {
  if (!desc || !k_tree || !v_tree || !k_cache || !v_cache || !path || !accept_len || !prefix_len)
    return JK_ERR_INVALID_ARG;
  const jk_attn_desc& d = *desc;
  if (d.batch < 1 || d.n_tree < 1 || d.n_tree > JK_MAX_TREE || d.n_kv_heads < 1 || d.head_dim < 1)
    return JK_ERR_INVALID_ARG;
  if (d.dtype != JK_BF16 && d.dtype != JK_F32) return JK_ERR_INVALID_ARG;
  if (max_depth < 1 || cache_capacity < 1) return JK_ERR_INVALID_ARG;
  if ((long long)d.batch * max_depth > 0x7fffffffLL || n_layers > 65535) return JK_ERR_UNSUPPORTED;
  const int64_t es = d.dtype == JK_BF16 ? 2 : 4;
  const int64_t align = 16 / es;  // elements per 16-byte chunk
  if (d.head_dim % align) return JK_ERR_UNSUPPORTED;
  const int64_t strides[] = {d.kc_stride_b, d.kc_stride_l, d.kc_stride_h, d.kt_stride_b, d.kt_stride_t, d.kt_stride_h};
  for (int64_t s : strides)
    if (s < 0 || s % align) return JK_ERR_INVALID_ARG;
  if (n_layers == 0) {  // (with several layers the tensor pointers live on the device and cannot be checked here)
    const void* ptrs[] = {k_tree, v_tree, k_cache, v_cache};
    for (const void* p : ptrs)
      if (reinterpret_cast<uintptr_t>(p) % 16) return JK_ERR_INVALID_ARG;
  }
  if (pages) {
    if (!pages->block_table || pages->page_size < 1 || pages->max_blocks < 1 || pages->n_pages < 1)
      return JK_ERR_INVALID_ARG;
    if (pages->page_stride < 0 || pages->page_stride % align) return JK_ERR_INVALID_ARG;
    if ((long long)pages->max_blocks * pages->page_size < cache_capacity) return JK_ERR_INVALID_ARG;
  }
  CommitArgs a;
  a.d = d;
  a.k_tree = k_tree; a.v_tree = v_tree; a.k_cache = k_cache; a.v_cache = v_cache;
  a.path = path; a.accept_len = accept_len; a.prefix_len = prefix_len;
  a.max_depth = max_depth; a.capacity = cache_capacity; a.advance = advance != 0;
  a.n_layers = n_layers;
  a.block_table = pages ? pages->block_table : nullptr;
  a.max_blocks = pages ? pages->max_blocks : 0;
  a.page_size = pages ? pages->page_size : 0;
  a.n_pages = pages ? pages->n_pages : 0;
  a.page_stride = pages ? pages->page_stride : 0;
  return launch_commit(a, static_cast<hipStream_t>(hip_stream)) == hipSuccess ? JK_OK : JK_ERR_HIP;
}

jk_status jk_commit_path(const jk_attn_desc* desc, const void* k_tree, const void* v_tree, void* k_cache,
                         void* v_cache, const int32_t* path, const int32_t* accept_len, int32_t max_depth,
                         int32_t cache_capacity, int32_t* prefix_len, int32_t advance, void* hip_stream) {
  return commit_common(desc, nullptr, 0, k_tree, v_tree, k_cache, v_cache, path, accept_len, max_depth,
                       cache_capacity, prefix_len, advance, hip_stream);
}

jk_status jk_commit_path_layers(const jk_attn_desc* desc, int32_t n_layers, const void* const* k_tree,
                                const void* const* v_tree, void* const* k_cache, void* const* v_cache,
                                const int32_t* path, const int32_t* accept_len, int32_t max_depth,
                                int32_t cache_capacity, int32_t* prefix_len, int32_t advance, void* hip_stream) {
  if (n_layers < 1) return JK_ERR_INVALID_ARG;
  return commit_common(desc, nullptr, n_layers, k_tree, v_tree,
                       const_cast<void**>(reinterpret_cast<void* const*>(k_cache)),
                       const_cast<void**>(reinterpret_cast<void* const*>(v_cache)), path, accept_len, max_depth,
                       cache_capacity, prefix_len, advance, hip_stream);
}

jk_status jk_commit_path_layers_paged(const jk_attn_desc* desc, const jk_paged_kv* pages, int32_t n_layers,
                                      const void* const* k_tree, const void* const* v_tree, void* const* k_pool,
                                      void* const* v_pool, const int32_t* path, const int32_t* accept_len,
                                      int32_t max_depth, int32_t* prefix_len, int32_t advance, void* hip_stream) {
  if (n_layers < 1 || !pages) return JK_ERR_INVALID_ARG;
  const long long cap = (long long)pages->max_blocks * pages->page_size;
  return commit_common(desc, pages, n_layers, k_tree, v_tree,
                       const_cast<void**>(reinterpret_cast<void* const*>(k_pool)),
                       const_cast<void**>(reinterpret_cast<void* const*>(v_pool)), path, accept_len, max_depth,
                       (int32_t)(cap > 0x7fffffffLL ? 0x7fffffffLL : cap), prefix_len, advance, hip_stream);
}

size_t jk_draft_heads_workspace(int32_t rows, int32_t d_model, int32_t vocab) {
  if (!heads_shape_ok(rows, d_model, vocab)) return 0;
  return most_bytes(rows, [&](int r) { return draft_heads_workspace_bytes(r, d_model, vocab); });
}

jk_status jk_draft_heads(const jk_draft_heads_desc* desc, const void* f_top, const float* s_top,
                         const void* w_head, float* logits, float* draft_probs, int32_t* topk_tokens,
                         float* topk_probs, void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!desc || !f_top || !s_top || !w_head || !logits || !topk_tokens || !topk_probs) return JK_ERR_INVALID_ARG;
  const jk_draft_heads_desc& d = *desc;
  if (d.rows < 1 || d.d_model < 1 || d.vocab < 1 || d.top_k < 1 || d.top_k > d.vocab) return JK_ERR_INVALID_ARG;
  if (d.mode != JK_HEADS_DECOUPLED && d.mode != JK_HEADS_CONTRASTIVE) return JK_ERR_INVALID_ARG;
  if (!(d.temperature > 0.f) || !std::isfinite(d.temperature)) return JK_ERR_INVALID_ARG;
  if (d.mode == JK_HEADS_CONTRASTIVE && (!std::isfinite(d.alpha) || !std::isfinite(d.beta))) return JK_ERR_INVALID_ARG;
  if (reinterpret_cast<uintptr_t>(f_top) % 16 || reinterpret_cast<uintptr_t>(w_head) % 16) return JK_ERR_INVALID_ARG;
  if (d.rows > 128 || d.d_model < 128 || d.d_model > 16384 || d.d_model % 128 || d.top_k > 16) return JK_ERR_UNSUPPORTED;
  if ((long long)2 * d.rows * d.vocab > 0x7fffffffLL * 4) return JK_ERR_UNSUPPORTED;
  if (d.vocab > (1 << 24)) return JK_ERR_UNSUPPORTED;
  const size_t need = draft_heads_least_bytes(d.rows, d.d_model, d.vocab);
  if (!workspace || reinterpret_cast<uintptr_t>(workspace) % 256 || workspace_bytes < need) return JK_ERR_WORKSPACE;
  DraftHeadsArgs a;
  a.rows = d.rows; a.d_model = d.d_model; a.vocab = d.vocab; a.top_k = d.top_k; a.mode = d.mode;
  a.temperature = d.temperature; a.alpha = d.alpha; a.beta = d.beta;
  a.f_top = f_top; a.w_head = w_head; a.s_top = s_top;
  a.logits = logits; a.draft_probs = draft_probs; a.topk_probs = topk_probs; a.topk_tokens = topk_tokens;
  a.workspace = workspace;
  a.workspace_bytes = workspace_bytes;
  return launch_draft_heads(a, static_cast<hipStream_t>(hip_stream)) == hipSuccess ? JK_OK : JK_ERR_HIP;
}

size_t jk_moe_experts_workspace(const jk_moe_desc* desc) {
  if (!desc || !moe_desc_ok(*desc) || !moe_desc_supported(*desc)) return 0;
  return most_bytes(desc->rows, [&](int r) { return moe_experts_workspace_bytes(r, desc->d_model, desc->d_ff, desc->n_experts); });
}

jk_status jk_moe_experts(const jk_moe_desc* desc, const void* u, const void* centroids, const void* w_gate,
                         const void* w_up, const void* w_down, void* f_top, float* s_top, int32_t* expert_idx,
                         void* f_mix, void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!desc || !u || !centroids || !w_gate || !w_up || !w_down || !f_top || !s_top || !expert_idx)
    return JK_ERR_INVALID_ARG;
  if (!moe_desc_ok(*desc)) return JK_ERR_INVALID_ARG;
  for (const void* ptr : {u, centroids, w_gate, w_up, w_down, (const void*)f_top, (const void*)f_mix})
    if (reinterpret_cast<uintptr_t>(ptr) % 16) return JK_ERR_INVALID_ARG;
  if (!moe_desc_supported(*desc)) return JK_ERR_UNSUPPORTED;
  const size_t need = moe_experts_workspace_bytes(desc->rows, desc->d_model, desc->d_ff, desc->n_experts);
  if (!workspace || reinterpret_cast<uintptr_t>(workspace) % 256 || workspace_bytes < need) return JK_ERR_WORKSPACE;
  MoeArgs a;
  a.rows = desc->rows; a.d_model = desc->d_model; a.d_ff = desc->d_ff; a.n_experts = desc->n_experts;
  a.u = u; a.centroids = centroids; a.w_gate = w_gate; a.w_up = w_up; a.w_down = w_down;
  a.f_top = f_top; a.f_mix = f_mix; a.s_top = s_top; a.expert_idx = expert_idx; a.workspace = workspace;
  return launch_moe_experts(a, static_cast<hipStream_t>(hip_stream)) == hipSuccess ? JK_OK : JK_ERR_HIP;
}

static bool tree_state_ok(const jk_tree_state* s) {
  return s && s->tokens && s->parent && s->score && s->q_row && s->n_nodes && s->max_nodes >= 1;
}

jk_status jk_tree_grow(const jk_tree_state* state, int32_t batch, int32_t n_front, int32_t top_k, int32_t width,
                       int32_t q_row_base, const int32_t* frontier_in, const int32_t* cand_tokens,
                       const float* cand_probs, int32_t* frontier_out, void* hip_stream) {
  if (!tree_state_ok(state) || !cand_tokens || !cand_probs || !frontier_out) return JK_ERR_INVALID_ARG;
  if (batch < 1 || n_front < 1 || top_k < 1 || width < 1 || q_row_base < 0) return JK_ERR_INVALID_ARG;
  if (!frontier_in && n_front != 1) return JK_ERR_INVALID_ARG;
  if (state->max_nodes > tree_max_nodes() || (long long)n_front * 2 * top_k > 256 || width > 256 || batch > 65535)
    return JK_ERR_UNSUPPORTED;
  TreeGrowArgs a;
  a.batch = batch; a.n_front = n_front; a.top_k = top_k; a.width = width; a.max_nodes = state->max_nodes;
  a.q_row_base = q_row_base;
  a.tokens = state->tokens; a.parent = state->parent; a.q_row = state->q_row; a.n_nodes = state->n_nodes;
  a.score = state->score;
  a.frontier_in = frontier_in; a.cand_tok = cand_tokens; a.cand_p = cand_probs; a.frontier_out = frontier_out;
  a.mg_top_k = 65536u / (unsigned)top_k + 1u;
  return launch_tree_grow(a, static_cast<hipStream_t>(hip_stream)) == hipSuccess ? JK_OK : JK_ERR_HIP;
}

jk_status jk_tree_grow_tail(const jk_tree_state* state, int32_t batch, int32_t n_front, int32_t top_k, int32_t k1,
                            int32_t k2, int32_t width, int32_t q_row_base, const int32_t* frontier_in,
                            const int32_t* cand_tokens, const float* cand_probs, void* hip_stream) {
  if (!tree_state_ok(state) || !cand_tokens || !cand_probs) return JK_ERR_INVALID_ARG;
  if (batch < 1 || n_front < 1 || top_k < 1 || k1 < 1 || k2 < 1 || k1 > top_k || k2 > top_k || width < 1 ||
      q_row_base < 0)
    return JK_ERR_INVALID_ARG;
  if (!frontier_in && n_front != 1) return JK_ERR_INVALID_ARG;
  if (state->max_nodes > tree_max_nodes() || (long long)n_front * k1 > 256 || (long long)width * k2 > 256 ||
      batch > 65535)
    return JK_ERR_UNSUPPORTED;
  TreeGrowArgs a;
  a.batch = batch; a.n_front = n_front; a.top_k = top_k; a.width = width; a.max_nodes = state->max_nodes;
  a.q_row_base = q_row_base;
  a.tokens = state->tokens; a.parent = state->parent; a.q_row = state->q_row; a.n_nodes = state->n_nodes;
  a.score = state->score;
  a.frontier_in = frontier_in; a.cand_tok = cand_tokens; a.cand_p = cand_probs; a.frontier_out = nullptr;
  return launch_tree_grow_tail(a, k1, k2, static_cast<hipStream_t>(hip_stream)) == hipSuccess ? JK_OK : JK_ERR_HIP;
}

jk_status jk_tree_fill_static(const jk_tree_state* state, int32_t batch, int32_t n_front, int32_t top_k,
                              int32_t q_row_base, const int32_t* frontier_in, const int32_t* cand_tokens,
                              const float* cand_probs, const int32_t* shape_slot, const int32_t* shape_expert,
                              const int32_t* shape_rank, int32_t n_new, const int32_t* next_index, int32_t n_next,
                              int32_t* frontier_out, int32_t* new_ids, void* hip_stream) {
  if (!tree_state_ok(state) || !cand_tokens || !cand_probs || !shape_slot || !shape_expert || !shape_rank)
    return JK_ERR_INVALID_ARG;
  if (batch < 1 || n_front < 1 || top_k < 1 || n_new < 1 || n_next < 0 || q_row_base < 0) return JK_ERR_INVALID_ARG;
  if (!frontier_in && n_front != 1) return JK_ERR_INVALID_ARG;
  if (n_next > 0 && (!next_index || !frontier_out)) return JK_ERR_INVALID_ARG;
  if (state->max_nodes > tree_max_nodes() || n_new > 4096 || n_next > 4096 || batch > 65535) return JK_ERR_UNSUPPORTED;
  TreeGrowArgs a;
  a.batch = batch; a.n_front = n_front; a.top_k = top_k; a.width = n_next; a.max_nodes = state->max_nodes;
  a.q_row_base = q_row_base;
  a.tokens = state->tokens; a.parent = state->parent; a.q_row = state->q_row; a.n_nodes = state->n_nodes;
  a.score = state->score;
  a.frontier_in = frontier_in; a.cand_tok = cand_tokens; a.cand_p = cand_probs;
  a.frontier_out = n_next > 0 ? frontier_out : nullptr;
  return launch_tree_fill_static(a, shape_slot, shape_expert, shape_rank, n_new, next_index, n_next, new_ids,
                                 static_cast<hipStream_t>(hip_stream)) == hipSuccess
             ? JK_OK
             : JK_ERR_HIP;
}

jk_status jk_tree_finalize(const jk_tree_state* state, int32_t batch, int32_t n_keep, int32_t* tree_tokens,
                           int32_t* parent, int32_t* q_row, int32_t* old_index, int32_t* n_valid, void* hip_stream) {
  if (!tree_state_ok(state) || !tree_tokens || !parent || !q_row || !n_valid) return JK_ERR_INVALID_ARG;
  if (batch < 1 || n_keep < 1 || n_keep > state->max_nodes) return JK_ERR_INVALID_ARG;
  if (state->max_nodes > tree_max_nodes() || batch > 65535) return JK_ERR_UNSUPPORTED;
  TreeFinalArgs a;
  a.batch = batch; a.n_keep = n_keep; a.max_nodes = state->max_nodes;
  a.tokens = state->tokens; a.parent = state->parent; a.q_row = state->q_row; a.n_nodes = state->n_nodes;
  a.score = state->score;
  a.out_tokens = tree_tokens; a.out_parent = parent; a.out_q_row = q_row; a.out_old = old_index; a.n_valid = n_valid;
  return launch_tree_finalize(a, static_cast<hipStream_t>(hip_stream)) == hipSuccess ? JK_OK : JK_ERR_HIP;
}

jk_status jk_gather_draft_probs(int32_t batch, int32_t n_tree, int32_t vocab, const float* q_all, int64_t n_q_rows,
                                const int32_t* q_row, float* draft_probs, void* hip_stream) {
  if (!q_all || !q_row || !draft_probs || batch < 1 || n_tree < 1 || vocab < 1 || n_q_rows < 1)
    return JK_ERR_INVALID_ARG;
  if ((long long)batch * n_tree > 0x7fffffffLL) return JK_ERR_UNSUPPORTED;
  return launch_gather_rows(q_all, q_row, draft_probs, (long long)batch * n_tree, vocab, n_q_rows,
                            static_cast<hipStream_t>(hip_stream)) == hipSuccess
             ? JK_OK
             : JK_ERR_HIP;
}

size_t jk_linear_workspace(int32_t m, int32_t n, int32_t k) {
  if (!linear_shape_ok(m, n, k)) return 0;
  return most_bytes(m, [&](int r) { return linear_workspace_bytes(r, n, k); });
}

jk_status jk_linear(int32_t m, int32_t n, int32_t k, const void* x, const void* w, const void* residual,
                    void* out_bf16, float* out_f32, void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (jk_status s = linear_refused(m, n, k, x, w, out_bf16, out_f32); s != JK_OK) return s;
  if (!workspace || reinterpret_cast<uintptr_t>(workspace) % 256 || workspace_bytes < linear_workspace_bytes(m, n, k))
    return JK_ERR_WORKSPACE;
  return linear_launched(m, n, k, x, w, residual, out_bf16, out_f32, workspace, hip_stream);
}

jk_status jk_workspace_init(void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!workspace || reinterpret_cast<uintptr_t>(workspace) % 256) return JK_ERR_WORKSPACE;
  return launch_zero_fill(workspace, workspace_bytes, static_cast<hipStream_t>(hip_stream)) == hipSuccess
             ? JK_OK
             : JK_ERR_HIP;
}

jk_status jk_stream_read_probe(const void* src, size_t bytes, void* sink, void* hip_stream) {
  if (!src || !sink || reinterpret_cast<uintptr_t>(src) % 16) return JK_ERR_INVALID_ARG;
  return launch_stream_read(src, bytes, sink, static_cast<hipStream_t>(hip_stream)) == hipSuccess ? JK_OK
                                                                                                  : JK_ERR_HIP;
}

jk_status jk_init(void* hip_stream) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return JK_ERR_HIP;
  bool rr = false;
  if (probe_xcd_placement(static_cast<hipStream_t>(hip_stream), &rr) != hipSuccess) return JK_ERR_HIP;
  g_xcd_state[dev] = rr ? 1 : 2;
  return JK_OK;
}

jk_status jk_set_tuning(const char* name, int32_t value) {
  if (!name) return JK_ERR_INVALID_ARG;
  Tuning& t = tuning();
  const struct { const char* name; int* field; } table[] = {
      {"attn_wm", &t.attn_wm}, {"attn_wn", &t.attn_wn}, {"attn_splits", &t.attn_splits},
      {"attn_fused", &t.attn_fused}, {"attn_deep", &t.attn_deep}, {"accept_single", &t.accept_single}, {"spin_limit", &t.spin_limit},
      {"ring_gemm", &t.ring_gemm}, {"narrow_gemm", &t.narrow_gemm}, {"verbose", &t.verbose}};
  for (const auto& e : table)
    if (std::strcmp(name, e.name) == 0) {
      *e.field = value;
      return JK_OK;
    }
  return JK_ERR_INVALID_ARG;
}

int32_t jk_last_device_error(const void* workspace) {
  if (!workspace) return -1;
  unsigned word = 0;
  if (hipMemcpy(&word, workspace, sizeof(word), hipMemcpyDeviceToHost) != hipSuccess) return -1;
  return (int32_t)(word & 0x7fffffffu);
}

jk_status jk_validate_tree(const int32_t* parent_host, int32_t n_tree) {
  if (!parent_host || n_tree < 1 || n_tree > JK_MAX_TREE) return JK_ERR_INVALID_ARG;
  for (int32_t i = 0; i < n_tree; ++i)
    if (parent_host[i] < -1 || parent_host[i] >= i) return JK_ERR_BAD_TREE;
  return JK_OK;
}

const char* jk_status_string(int32_t status) {
  switch (status) {
    case JK_OK: return "ok";
    case JK_ERR_INVALID_ARG: return "invalid argument";
    case JK_ERR_BAD_TREE: return "parent[] violates -1 <= parent[i] < i";
    case JK_ERR_UNSUPPORTED: return "unsupported shape";
    case JK_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case JK_ERR_HIP: return "HIP runtime error";
    case JK_ERR_SCRATCH_LIMIT: return "input too large for the library's built-in scratch buffer";
    default: return "unknown status";
  }
}

const char* jk_version(void) { return "0.1"; }

}  // extern "C"
