// Products of few rows with large weight matrices (gfx950), Y[M, N] = X[M, K] . W[N, K]^T, bf16 operands, fp32
// accumulation: the output heads and the experts' projections of up to 32 rows (an expert's rows in blocks of so many).
//
// What bounds it: the weight stream.  stream_gemm.hip gives every workgroup a strip of 128 weight rows, which leaves CUs idle in
// the last turn of workgroups and wherever there are fewer strips than CUs.  Here a workgroup per CU has an equal share of all
// weight rows, counted in groups of 16, whichever expert they belong to, and goes through it in batches of a few groups and all
// of k.  A wave has every fourth 64 of k: 128 bytes of a batch's weight rows and of X's rows come straight into its own ring in
// LDS (global_load_lds_dwordx4), two or more such units ahead, across the ends of batches and experts; the four waves' sums are
// added up in LDS at the end of a batch while the next one's first units arrive.  X is drawn from the L2 once per batch, which
// is why a batch has several groups: a CU draws about 51 bytes per ns, HBM's share is 22 - 25.
// Measured (us, all kernels of a call, strips of 128 rows / this): heads of 2 rows, 69951 x 2944 96.3 / 82.6, 34482 x 1280 37.3 /
// 27.5; 28 rows, 23879 x 2560 39.9 / 34.5; 30 rows, 47383 x 7424 158.5 / 142.5; experts of 1 row, two of five of 2944 x 3200 61.1 /
// 36.2; 7 rows, eight of 4736 x 2816 146.6 / 123.9; 49 rows, eight of 1920 x 10496 202.7 / 186.2.  Where strips fill their turns
// they are as fast or faster (20 rows, 128256 x 4096 195 / 205; 40 rows, eight experts of 4096 x 4096 151 / 153): rows a power of
// two apart meet in the same memory channels, and a batch's unit is 64 or more of them at once.  Tried and no faster: the
// weights straight into registers in the matrix operands' layout (205), other orders of batches and of k (204 - 232), one to four
// units in flight (205 - 207), X left out (207).
#include <type_traits>

#include "jk_device.h"
#include "jk_internal.h"
#include "ring_share.h"
#include "xcd_grid.h"

namespace jk {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// What is computed:
//   HEADS  logits of the rows that the two output heads see, made of the tokens' two features as they are taken from LDS
//          (see StreamGemmArgs)
//   PAIR   act = silu(gate) * up of the rows that chose an expert; a group has eight gate rows and the same of the up projection
//   DOWN   the expert's output projection, of the rows it has
enum RingKind { HEADS, PAIR, DOWN };

constexpr int kWaves = 4, kRingThreads = 64 * kWaves, kUnit = 64;  // a unit: 64 of k
constexpr int kMaxRows = 128, kMaxRingExperts = 64, kMaxItems = kMaxRingExperts + 2 * kMaxRows / 8;

// RG: groups of eight rows of X, NF: groups of 16 weight rows in a batch
template <RingKind KIND, int RG, int NF>
struct RingCfg {
  static constexpr int MT = (RG + 1) / 2;
  static constexpr int PER = 2 * NF + RG;            // transfers of a unit, 8 rows of 128 bytes each
  static constexpr int QUADS = NF * 4, PITCH = QUADS + 1;  // of a row of sums (and a quad against bank conflicts)
  static constexpr int SUMS = 2 * 16 * MT * PITCH * 16;
  static constexpr int LISTS = KIND == HEADS ? 0 : 2 * kMaxRows * 4 + kMaxRingExperts * 8 + kMaxItems * 4 + 16;
  static constexpr int FIT = (160 * 1024 - SUMS - LISTS - 1024) / (kWaves * PER * 1024), MOST = 63 / PER + 1;
  static constexpr int WANT = FIT < MOST ? FIT : MOST, DEPTH = WANT < 6 ? WANT : 6;  // units in flight
  static constexpr int RING = DEPTH * PER * 1024;    // bytes of a wave
  static constexpr int SMEM = kWaves * RING + 1024 + SUMS + LISTS;  // (1024: the rows that the last 16 of X may lack)
  static_assert(DEPTH >= 2, "LDS plan");
};

// (The leading arguments are in scalar registers when a wave starts, see stream_gemm.hip)
template <RingKind KIND, int RG, int NF>
__global__ __launch_bounds__(kRingThreads, 1) void ring_gemm_kernel(const int* sel_lead, int rows_all, int experts, int n, int k, int all,
                                                                    const uint16_t* x, const uint16_t* w, long long w_batch, StreamGemmArgs p) {
  p.sel = sel_lead;
  p.m = rows_all;
  p.batch = experts;
  p.n = n;
  p.k = k;
  p.x = x;
  p.w = w;
  p.w_batch = w_batch;
  using C = RingCfg<KIND, RG, NF>;
  constexpr int MT = C::MT, CAP = 8 * RG, GROUP = KIND == PAIR ? 8 : 16;  // rows of X at a time; output columns of a group
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), r = lane & 15, g = lane >> 4;
  unsigned char* ring = smem + wave * C::RING;
  const unsigned ring_at = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)ring;
  floatx4* sums = reinterpret_cast<floatx4*>(smem + kWaves * C::RING + 1024);  // [2][CAP][PITCH]
  int* order = reinterpret_cast<int*>(smem + kWaves * C::RING + 1024 + C::SUMS);  // the choices, expert by expert: 2 row + (first or second)
  int* starts = order + 2 * kMaxRows;       // where an expert's begin
  int* counts = starts + kMaxRingExperts;   // and how many it has
  int* item_s = counts + kMaxRingExperts;   // (expert, block of CAP rows) pairs that there is something to do for; and how many of them

  // ---- items: the experts that somebody chose, each with up to CAP rows of X at a time.  One wave finds them, a lane per row and
  // per expert: a bit per row and expert in LDS, counted.  (Expert by expert, in every wave, it took 0.15 us of each: a launch for eight
  // experts 1.2 us less like this, 9 rows and 64 experts of 768 x 256 44.0 -> 25.7 us.)
  int items = 1;
  if constexpr (KIND != HEADS) {
    if (wave == 0) {
      uint4* chosen = reinterpret_cast<uint4*>(order);  // [expert]: bit r: row r chose it (what is read here is read before the order is written)
      auto in_order = [] { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); };  // (LDS operations of a wave complete in order)
      const int2* sel = reinterpret_cast<const int2*>(p.sel);
      const int2 none = make_int2(-1, -1), s0 = lane < p.m ? sel[lane] : none, s1 = lane + 64 < p.m ? sel[lane + 64] : none;
      const int e[4] = {s0.x, s0.y, s1.x, s1.y};
      chosen[lane] = make_uint4(0u, 0u, 0u, 0u);
      in_order();
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if ((unsigned)e[c] < (unsigned)p.batch) atomicOr(reinterpret_cast<unsigned*>(chosen + e[c]) + 2 * (c >> 1) + (lane >> 5), 1u << (lane & 31));
      in_order();
      auto bits = [](unsigned lo, unsigned hi) { return (unsigned long long)hi << 32 | lo; };
      const unsigned long long below = (1ull << lane) - 1ull;
      int rank[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const uint4 v = chosen[(unsigned)e[c] < (unsigned)p.batch ? e[c] : 0];
        rank[c] = c < 2 ? __popcll(bits(v.x, v.y) & below) : __popcll(bits(v.x, v.y)) + __popcll(bits(v.z, v.w) & below);
      }
      const uint4 own = chosen[lane];
      const int rows = __popcll(bits(own.x, own.y)) + __popcll(bits(own.z, own.w)), blocks = (rows + CAP - 1) / CAP;
      int upto = rows | blocks << 16;  // sums over the experts up to this lane's: rows at most 256, blocks at most kMaxItems
      auto add = [&](int v) { upto += v; };
      add(__builtin_amdgcn_update_dpp(0, upto, 0x111, 0xf, 0xf, false));  // row_shr:1, 2, 4, 8
      add(__builtin_amdgcn_update_dpp(0, upto, 0x112, 0xf, 0xf, false));
      add(__builtin_amdgcn_update_dpp(0, upto, 0x114, 0xf, 0xf, false));
      add(__builtin_amdgcn_update_dpp(0, upto, 0x118, 0xf, 0xf, false));
      add(__builtin_amdgcn_update_dpp(0, upto, 0x142, 0xa, 0xf, false));  // row_bcast:15 into rows 1 and 3
      add(__builtin_amdgcn_update_dpp(0, upto, 0x143, 0xc, 0xf, false));  // row_bcast:31 into rows 2 and 3
      starts[lane] = (upto & 0xffff) - rows;
      counts[lane] = rows;
      if (lane == 63) item_s[kMaxItems] = upto >> 16;
      for (int b = 0; b < blocks; ++b) item_s[(upto >> 16) - blocks + b] = lane | b << 8;
      in_order();
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if ((unsigned)e[c] < (unsigned)p.batch) order[starts[e[c]] + rank[c]] = 2 * (lane + 64 * (c >> 1)) + (c & 1);
    }
    __syncthreads();
    items = __builtin_amdgcn_readfirstlane(item_s[kMaxItems]);
  }

  // ---- this workgroup's share of the groups (neighbours on one XCD have the same X)
  const int blk = blockIdx.x;
  const int id = xcd_place(blk, all);
  const int per_item = (p.n + GROUP - 1) / GROUP;
  const ring::Shares shares{per_item, NF};
  const int f0 = (int)shares.share_begin(items, id, all), f1 = (int)shares.share_begin(items, id + 1, all);
  if (f0 == f1) return;  // (the whole workgroup)
  auto expert_of = [&](int item) { return KIND == HEADS ? 0 : __builtin_amdgcn_readfirstlane(item_s[item]) & 255; };
  auto block_of = [&](int item) { return KIND == HEADS ? 0 : __builtin_amdgcn_readfirstlane(item_s[item]) >> 8; };
  auto rows_of = [&](int item) { return KIND == HEADS ? p.m : __builtin_amdgcn_readfirstlane(counts[expert_of(item)]) - block_of(item) * CAP; };

  // ---- the asking side: where the next unit comes from
  const int lrow = lane >> 3, lcol = 16 * ((lane & 7) ^ lrow);  // (a transfer's row and, swizzled, its chunk of it)
  const int units = p.k / kUnit, count = (units - wave + kWaves - 1) / kWaves;  // this wave's units of a batch
  // (workgroups start at different units: rows often lie a power of two apart, in step all would ask the same few channels)
  const int rot = count > 0 ? (int)((5u * blk + (blk >> 3)) % (unsigned)count) : 0;
  const uint16_t *wa, *wb, *xa;  // of the batch that is asked for: the weights (PAIR: gate and up) and X
  unsigned wr[2 * NF], xr[RG];
  auto aim_x = [&](int item) {
    const int e = expert_of(item), first = block_of(item) * CAP, rows = rows_of(item);
    xa = dev::uniform_ptr(p.x);
#pragma unroll
    for (int i = 0; i < RG; ++i) {  // (rows past the end repeat the last one; never stored)
      int row = min(8 * i + lrow, rows - 1);
      if constexpr (KIND != HEADS) row = order[starts[e] + first + row] >> (KIND == PAIR);
      xr[i] = (unsigned)row * (unsigned)p.k * 2u + lcol;
    }
  };
  auto aim_w = [&](const ring::Batch& b) {
    const long long at = (long long)expert_of(b.item) * p.w_batch + (long long)b.off * GROUP * p.k;
    wa = dev::uniform_ptr(p.w + at);
    if constexpr (KIND == PAIR) wb = dev::uniform_ptr(p.w2 + at);
    const int last = min(b.size * GROUP, p.n - b.off * GROUP) - 1;
#pragma unroll
    for (int i = 0; i < (KIND == PAIR ? NF : 2 * NF); ++i) wr[i] = (unsigned)min(8 * i + lrow, last) * (unsigned)p.k * 2u + lcol;
  };
  ring::Batch asked = shares.first(f0, f1);
  int left_a = f1 - f0, ja = 0;  // groups from `asked` on, and its next unit
  ring::Batch used = asked;
  int left_u = left_a;
  bool more = count > 0;
  aim_x(asked.item);
  aim_w(asked);
  auto ask = [&](int slot) {
    const int u = ja + rot, at = (wave + kWaves * (u < count ? u : u - count)) * kUnit;
    const unsigned to = ring_at + slot * (C::PER * 1024);
#pragma unroll
    for (int i = 0; i < 2 * NF; ++i) {
      if constexpr (KIND == PAIR) dev::dma16((i & 1 ? wb : wa) + at, wr[i >> 1], to + 1024 * i);
      else dev::dma16(wa + at, wr[i], to + 1024 * i);
    }
#pragma unroll
    for (int i = 0; i < RG; ++i) dev::dma16(xa + at, xr[i], to + 1024 * (2 * NF + i));
    if (++ja == count) {
      ja = 0;
      left_a -= asked.size;
      more = left_a > 0;
      if (more) {
        const int was = asked.item;
        asked = shares.next(asked, left_a);
        if (asked.item != was) aim_x(asked.item);
        aim_w(asked);
      }
    }
  };

  // ---- HEADS: row 2 r + h of the left side from rows 2 r and 2 r + 1 as they lie in LDS (a term whose coefficient is zero is
  // left out, so that a NaN in the other expert's feature cannot leak into a decoupled head)
  const bool mixed = KIND == HEADS && p.heads_mode != JK_HEADS_DECOUPLED;
  float c_own[MT], c_other[MT];
  if constexpr (KIND == HEADS) {
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      const int row = min(16 * t + r, p.m - 1);  // (p.m is even: a row past the end has a partner past the end)
      const float s_own = p.s_top[row], s_other = p.s_top[row ^ 1];
      c_own[t] = mixed && (row & 1) ? -p.alpha : s_own;
      c_other[t] = !mixed ? 0.f : (row & 1) ? p.beta : s_other;
    }
  }
  auto mix = [&](bf16x8 v, int t) {
    const u32x4 x = __builtin_bit_cast(u32x4, v);
    const unsigned keep = c_own[t] != 0.f ? ~0u : 0u, keep_other = c_other[t] != 0.f ? ~0u : 0u;
    u32x4 o;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const unsigned own = x[j] & keep;
      float lo = c_own[t] * __uint_as_float(own << 16), hi = c_own[t] * __uint_as_float(own & 0xFFFF0000u);
      if (mixed) {
        const unsigned other = (unsigned)__builtin_amdgcn_update_dpp(0, (int)x[j], 0xB1, 0xf, 0xf, true) & keep_other;  // (lane ^ 1)
        lo += c_other[t] * __uint_as_float(other << 16);
        hi += c_other[t] * __uint_as_float(other & 0xFFFF0000u);
      }
      o[j] = dev::pack_bf16(lo, hi);
    }
    return __builtin_bit_cast(bf16x8, o);
  };

  // ---- the stream
  floatx4 acc[NF][MT];
  auto clear = [&] {
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
      for (int t = 0; t < MT; ++t) acc[f][t] = floatx4{0.f, 0.f, 0.f, 0.f};
  };
  const int at0 = r * 128 + 16 * (g ^ (r & 7)), at1 = r * 128 + 16 * ((4 + g) ^ (r & 7));  // a lane's chunks of its row
  bf16x8 a[NF][2], b[MT][2];
  auto take = [&](int slot) {  // (and the slot may be filled again)
    const unsigned char* from = ring + slot * (C::PER * 1024);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
#pragma unroll
      for (int t = 0; t < MT; ++t) b[t][s] = *reinterpret_cast<const bf16x8*>(from + (2 * NF + 2 * t) * 1024 + (s ? at1 : at0));
#pragma unroll
      for (int f = 0; f < NF; ++f) a[f][s] = *reinterpret_cast<const bf16x8*>(from + 2 * f * 1024 + (s ? at1 : at0));
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  };
  auto multiply = [&] {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        const bf16x8 x = KIND == HEADS ? mix(b[t][s], t) : b[t][s];
#pragma unroll
        for (int f = 0; f < NF; ++f) acc[f][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[f][s], x, acc[f][t], 0, 0, 0);
      }
  };
  // (waits that stores of a batch's results make longer than they need be, never shorter)
  int in_flight = 0;
  auto wait_oldest = [&] {
    constexpr int D = C::DEPTH, P = C::PER;
    if (in_flight == D) dev::wait_vm<(D - 1) * P>();
    else if (D > 5 && in_flight == 5) dev::wait_vm<(D > 5 ? 4 * P : 0)>();
    else if (D > 4 && in_flight == 4) dev::wait_vm<(D > 4 ? 3 * P : 0)>();
    else if (D > 3 && in_flight == 3) dev::wait_vm<(D > 3 ? 2 * P : 0)>();
    else if (D > 2 && in_flight == 2) dev::wait_vm<(D > 2 ? P : 0)>();
    else dev::wait_vm<0>();
  };
  int to = 0, from = 0;  // slots
  auto ask_next = [&] {
    if (!more) return;
    ask(to);
    to = to + 1 == C::DEPTH ? 0 : to + 1;
    ++in_flight;
  };
#pragma unroll
  for (int i = 0; i < C::DEPTH; ++i) ask_next();

  for (;;) {
    clear();
    for (int j = 0; j < count; ++j) {
      wait_oldest();
      take(from);
      from = from + 1 == C::DEPTH ? 0 : from + 1;
      --in_flight;
      ask_next();
      multiply();
    }
    // ---- the waves' sums: two add the other two's to theirs, everybody adds those two up
    auto at = [&](int half, int f, int t) { return sums + (half * 16 * MT + 16 * t + r) * C::PITCH + 4 * f + g; };
    __syncthreads();  // (the sums of the batch before have been read)
    if (wave >= 2) {
#pragma unroll
      for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int t = 0; t < MT; ++t) *at(wave - 2, f, t) = acc[f][t];
    }
    __syncthreads();
    if (wave < 2) {
#pragma unroll
      for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int t = 0; t < MT; ++t) *at(wave, f, t) += acc[f][t];
    }
    __syncthreads();
    const int e = expert_of(used.item), first = block_of(used.item) * CAP, rows = min(rows_of(used.item), CAP);
    auto quad = [&](int row, int q) { return sums[row * C::PITCH + q] + sums[(16 * MT + row) * C::PITCH + q]; };
    if constexpr (KIND == PAIR) {
      const int per_row = used.size * 2;  // quads of gate rows
      for (int i = tid; i < rows * per_row; i += kRingThreads) {
        const int row = i / per_row, h = i - row * per_row, q = (h >> 1) * 4 + (h & 1);
        const floatx4 gate = quad(row, q), up = quad(row, q + 2);
        float o[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] = gate[j] / (1.f + expf(-gate[j])) * up[j];
        *reinterpret_cast<uint2*>(p.act + (long long)order[starts[e] + first + row] * p.n + used.off * GROUP + 4 * h) =
            make_uint2(dev::pack_bf16(o[0], o[1]), dev::pack_bf16(o[2], o[3]));
      }
    } else {
      const int per_row = used.size * 4, n0 = used.off * GROUP;
      float* y = p.y + n0;
      auto place = [&](int row) { return (long long)(KIND == DOWN ? order[starts[e] + first + row] : row); };
      if (KIND == DOWN || ((p.n & 3) == 0 && (reinterpret_cast<size_t>(p.y) & 15) == 0)) {
        for (int i = tid; i < rows * per_row; i += kRingThreads) {
          const int row = i / per_row, q = i - row * per_row;
          if (n0 + 4 * q >= p.n) continue;
          const floatx4 v = quad(row, q);
          floatx4* dst = reinterpret_cast<floatx4*>(y + place(row) * p.n + 4 * q);
          if constexpr (KIND == HEADS) __builtin_nontemporal_store(v, dst);
          else *dst = v;
        }
      } else {
        for (int i = tid; i < rows * per_row; i += kRingThreads) {
          const int row = i / per_row, q = i - row * per_row;
          const floatx4 v = quad(row, q);
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (n0 + 4 * q + j < p.n) y[(long long)row * p.n + 4 * q + j] = v[j];
        }
      }
    }
    left_u -= used.size;
    if (left_u <= 0) break;
    used = shares.next(used, left_u);
  }
}

template <RingKind KIND, int RG, int NF>
hipError_t launch(const StreamGemmArgs& p, hipStream_t stream) {
  static LdsLimitRaised raised;
  constexpr int smem = RingCfg<KIND, RG, NF>::SMEM;
  if (hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(ring_gemm_kernel<KIND, RG, NF>), smem, raised); e != hipSuccess) return e;
  const long long groups = (long long)((p.n + (KIND == PAIR ? 7 : 15)) / (KIND == PAIR ? 8 : 16)) * p.batch;
  const int cus = device_cu_count();
  const int all = (int)(groups < cus ? groups : cus);
  return launch_kernel(ring_gemm_kernel<KIND, RG, NF>, dim3((unsigned)all), dim3(kRingThreads), smem, stream, p.sel, p.m, p.batch, p.n, p.k, all, p.x,
                     p.w, p.w_batch, p);
}
// `items`: how many experts are likely to be chosen
template <RingKind KIND, int RG>
hipError_t launch_batches(const StreamGemmArgs& p, int items, hipStream_t stream) {
  const int groups = (p.n + (KIND == PAIR ? 7 : 15)) / (KIND == PAIR ? 8 : 16) * items, each = (groups + device_cu_count() - 1) / device_cu_count();
  if (each <= 2) return launch<KIND, RG, 2>(p, stream);
  return each <= 4 ? launch<KIND, RG, 4>(p, stream) : launch<KIND, RG, 6>(p, stream);
}
template <RingKind KIND>
hipError_t launch_rows(const StreamGemmArgs& p, int rows, int items, hipStream_t stream) {
  switch ((rows + 7) / 8) {
    case 1: return launch_batches<KIND, 1>(p, items, stream);
    case 2: return launch_batches<KIND, 2>(p, items, stream);
    case 3: return launch_batches<KIND, 3>(p, items, stream);
    case 4: return launch_batches<KIND, 4>(p, items, stream);
    default: return hipErrorInvalidValue;
  }
}
// whether strips of 128 weight rows fill their turns of workgroups (the other kernel's)
bool strips_fill(int strips) {
  const int cus = device_cu_count(), turns = (strips + cus - 1) / cus;
  return strips >= 0.96 * turns * cus;
}
}  // namespace

// Against strips of 128 rows in turns of workgroups (stream_gemm.hip): where strips fill their turns there is little to gain, and a
// batch's end (three barriers, its first units, X once more) weighs the more the shorter k is.  Kernel times of 250 heads
// and 1400 calls of experts, drawn over 1 - 16 tokens, 1 - 80 rows, k 512 - 8192 and 512 - 14336 rows of weights (heads 128256); strips /
// this, geometric mean (least): heads of less than three quarters of a turn of strips 1.05 - 1.3 (0.93), of more than that
// 0.99 (0.88); with more turns 1.16 (0.95).  More than 16 logits rows below 42 rows of weights a CU: 0.96 (0.93), three of them.
bool ring_gemm_takes_heads(int m, int n) {
  const int cus = device_cu_count(), strips = (n + 127) / 128;
  if (tuning().ring_gemm >= 0) return tuning().ring_gemm > 0 && m <= kRingRows;
  if (m > kRingRows || n < (m <= 16 ? 32 : 42) * cus || strips_fill(strips)) return false;
  return strips < 0.75 * cus || strips > cus;
}
// Experts' projections.  Strips that may need another turn (of the experts that rows could choose at most) are slow, and so are strips of
// experts that nobody chose; experts of more than 32 rows have their weights gone through once per block of so many.  Each of
// the two launches goes by its own line.  Gate and up: 1.3 in the mean, with few rows and strips up to 2.7; one turn of 0.85 or
// more 1.0 (0.8); full turns of a k that 1024 divides 1.00 (40 rows, eight of 4096 x 4096: the call 150.6 us, by strips 150.1); many
// rows 1.1 - 1.3 where the strips would leave four fifths of the CUs without work and k is short, else 0.7 - 1.2.
bool ring_gemm_takes_pair(const RingExperts& x, int d_ff, int d_model) {
  const int cus = device_cu_count(), per = (d_ff + 63) / 64, strips = x.likely * per;
  if (tuning().ring_gemm >= 0) return tuning().ring_gemm > 0;
  if (x.many) return strips <= cus / 5 && d_model < 3072;
  // (rows of weights a power of two apart meet in the same memory channels, and here more of them at once)
  const bool turns = x.most * per > cus && !(strips_fill(x.most * per) && d_model % 1024 == 0);
  return x.mean <= 2.0 || turns || strips < 0.85 * cus;
}
// Output projection: a long k over few columns is divided by the strips' kernel, and not by this one: 0.8 (0.54) from 4096 on, 0.97 from
// 3072.  Elsewhere up to 0.85 of a turn 1.07 (0.76), beyond 0.95 (0.75); other turns 1.2 (0.95), experts of a row or so 1.25.
// Both lines and the calls' other kernels: 1.207 times as fast as strips alone, one call of a hundred 6 % slower; both projections on
// one kernel, by one line for both, 1.201 and 9 %.
bool ring_gemm_takes_down(const RingExperts& x, int d_model, int d_ff) {
  const int cus = device_cu_count(), per = (d_model + 127) / 128, strips = x.likely * per;
  if (tuning().ring_gemm >= 0) return tuning().ring_gemm > 0;
  if (x.many) return strips <= cus / 6 && d_ff <= 1024;
  return x.mean <= 2.0 || x.most * per > cus || (strips < 0.85 * cus && (strips > cus / 6 || d_ff <= 3072));
}
hipError_t launch_ring_gemm_heads(const StreamGemmArgs& p, hipStream_t stream) { return launch_rows<HEADS>(p, p.m, 1, stream); }
hipError_t launch_ring_gemm_pair(const StreamGemmArgs& p, int rows, int items, hipStream_t stream) { return launch_rows<PAIR>(p, rows, items, stream); }
hipError_t launch_ring_gemm_down(const StreamGemmArgs& p, int rows, int items, hipStream_t stream) { return launch_rows<DOWN>(p, rows, items, stream); }

}  // namespace jk
