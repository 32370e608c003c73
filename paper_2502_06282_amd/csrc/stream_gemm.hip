// Products of few rows with weight matrices (gfx950): the draft layer's linear layers, its experts' projections, and the
// output heads.  Y[M, N] = X[M, K] . W[N, K]^T, M <= 256, bf16 operands, fp32 accumulation.
//
// What bounds it: the weight stream, and for a few tens of megabytes the round trip to memory in front of it.  So a wave
// fetches its weights straight into registers in MFMA layout (v_mfma_f32_16x16x32_bf16: 16 rows of 64 bytes per
// instruction, the other half of each 128-byte line with the next k step), 8 KB of them in flight from the first
// cycle on, each register asked for again as soon as its last product is issued; only X goes through LDS, one chunk of k
// ahead of its use, shared by the workgroup's eight waves; one barrier per chunk.  Narrow strips (128 weight rows) and
// whole k ranges where that gives every CU a workgroup, k split into as many parts as it takes otherwise.
// Measured on an MI355X (weights cold, us): eight experts' gate and up projections of 4096 x 4096 98; 20 rows, 128256 x 4096
// 175 (6.0 TB/s), 80 rows 204; 32768 x 4096, 4 rows 47 (5.7 TB/s), 128 rows 63: with many rows a CU draws as many bytes of X
// from L2 as of weights.  With weights through LDS rings and strips of 512 rows the first two took 114 and 177 us.
// Non-temporal weight loads (-10 %), chunks of 512 and more weights in flight (no difference) were tried.
#include <cmath>
#include <type_traits>

#include "jk_device.h"
#include "jk_internal.h"
#include "jk_wave.h"
#include "xcd_grid.h"

namespace jk {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 512;  // 8 waves
constexpr int kListBytes = 512;  // the choices of an expert (at most 128), 2 row + (first or second)

__device__ __forceinline__ unsigned bf16_bits_rne(float f) {
  const unsigned u = __float_as_uint(f);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (u >> 16) | 0x40u;  // NaN stays NaN
  return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}
__device__ __forceinline__ float bf16_lo(unsigned w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(unsigned w) { return __uint_as_float(w & 0xFFFF0000u); }

// What a workgroup computes:
//   PLAIN  a strip of Y = X . W^T
//   PAIR   the same strip of two weight tensors (an expert's gate and up projections), for the rows of X that chose the
//          expert; with an undivided k range the epilogue applies silu(gate) * up
//   DOWN   a strip of an expert's output projection, for the rows it has
//   HEADS  as PLAIN, of the rows that the two output heads see: row 2 r + h is c f_(h + 1) + c' f_(2 - h) of token r's two
//          features, rows 2 r and 2 r + 1 of x, rounded to bf16 (see StreamGemmArgs)
enum Kind { PLAIN, PAIR, DOWN, HEADS };

// NF: 16-row weight fragments of a wave, side by side; a workgroup has a strip of 128 NF weight rows
constexpr int strip_rows(int nf) { return 128 * nf; }
// k steps of 32 whose weights are in flight: 64 KB per workgroup (what a CU turns over in a round trip)
constexpr int steps_ahead(int nf) { return nf == 1 ? 8 : (nf <= 3 ? 4 : 2); }

// One strip for up to 16 MT rows
template <int MT, int NF>
struct Cfg {
  static constexpr int AHEAD = steps_ahead(NF);
  static constexpr int KC = MT > 8 && AHEAD < 8 ? 128 : 256;  // k per chunk of X
  static constexpr int KS = KC / 32;  // MFMA k steps per chunk
  static constexpr int LDX = KC + 8;  // bf16 per LDS row: 16 bytes of padding spread the rows over the banks
  static constexpr int PIECES = MT * 16 * (KC / 8);           // 16-byte pieces of an X chunk
  static constexpr int XP = (PIECES + kThreads - 1) / kThreads;
  static constexpr int X_BYTES = MT * 16 * LDX * 2;
  static constexpr int SMEM = 2 * X_BYTES;
  static_assert(SMEM + kListBytes <= 160 * 1024, "LDS plan");
  static constexpr int LOOK = 7;      // products between an X operand's read from LDS and its use
};

// A wave's weights: its rows' addresses, and the fragments of the next AHEAD k steps in registers
template <int NF, Kind KIND>
struct Weights {
  static constexpr int AHEAD = steps_ahead(NF);
  const uint16_t* row[NF];
  bf16x8 a[NF][AHEAD];
  int k0, k1;        // this part's k range, in units of 128
  unsigned wg;

  __device__ __forceinline__ void start(const StreamGemmArgs& p, int strips, int n_base, int e, int wave, int r, int g) {
    // (64-bit divisions here were half of the 412 instructions in front of the first load: 2 - 4 % of a small call)
    k0 = 0;
    k1 = p.k;
    if (p.ksplit > 1) {
      const unsigned units = (unsigned)p.k / 128u, parts = (unsigned)p.ksplit;  // (at most 8192 and 64: the products fit)
      k0 = (int)(blockIdx.z * units / parts) * 128;
      k1 = (int)((blockIdx.z + 1u) * units / parts) * 128;
    }
    wg = blockIdx.x + strips * blockIdx.y;
    const uint16_t* base = (KIND == PAIR && wave >= 4 ? p.w2 : p.w) + (long long)e * p.w_batch;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const int n = min(n_base + 16 * f + r, p.n - 1);  // rows past the end repeat the last one; never stored
      row[f] = base + (long long)n * p.k + 8 * g;
    }
  }
  // (what lies past a half chunk at the end of the range is fetched from inside it and not used)
  __device__ __forceinline__ void load(int k, int slot) {
    k = min(k, k1 - 32);
#pragma unroll
    for (int f = 0; f < NF; ++f) a[f][slot] = *reinterpret_cast<const bf16x8*>(row[f] + k);
  }
  // Workgroups start at different chunks and wrap around: rows often lie a power of two apart, so that workgroups in
  // step would all ask the same few memory channels (16 x 4096 x 4096: 115 us in step, 98 us like this; 32000 x 4096:
  // 58 and 46).  Workgroups run on the eight XCDs in turn, so the start has to vary within every eighth of them too: by seven
  // chunks from one to the next and by eight from XCD to XCD where a row has 16 chunks of 256 or more, else by 41 and five (5 wg + wg / 8).  Of 28 pairs of
  // steps, 41 and five / seven and eight, kernels of a call, us: 20 rows, 128256 x 4096 195 / 190, 80, 32000 x 4096 69.3 / 68.6, 40, 64000 x
  // 8192 196 / 193, eight experts of 4096 x 4096 148.8 / 144.7; in eight chunks the other way round, 64000 x 2048 1 : 0.985, experts of 2048 x
  // 8192 1 : 0.976.  Seven divides the chunks of k = 7168 and 14336, whose workgroups of an XCD then share four and eight places to start
  // with seven, and have 28 and 32 with 41: the calls are the same to 0.8 %, or faster with seven (40 rows, four experts of 7168 x 4096 134.7 /
  // 133.7, of 4096 x 14336 252.0 / 252.1, eight of 7168 x 2048 138.1 / 137.0; heads of 64 rows, 20000 x 7168 87.4 / 86.9, of 40, 64000 x 7168 182.5 /
  // 182.5, of 60, 100000 x 7168 349.5 / 350.6).  Chunks of 128 (more than 128 rows, wide strips) went both ways, 160 rows of 83155 x 3968 221.4 / 226, of 32000 x
  // 4096 88.7 / 86.5, and keep 41 and five, with which none of them lost.  (A half chunk at the end stays last.)
  template <int KC>
  __device__ __forceinline__ int chunk(int c) const {
    const int whole = (k1 - k0) / KC;
    const int rot = whole > 0 ? (int)((KC == 256 && whole >= 16 ? 8u * (wg & 7u) + 7u * (wg >> 3) : 5u * wg + (wg >> 3)) % (unsigned)whole) : 0;
    const int t = c + rot;
    return k0 + (c < whole ? (t < whole ? t : t - whole) : c) * KC;
  }
};

template <int MT, int NF, Kind KIND>
__device__ __forceinline__ void strip_products(const StreamGemmArgs& p, Weights<NF, KIND>& w, int m, const int* list, unsigned char* xbuf,
                                               int e) {
  using C = Cfg<MT, NF>;
  constexpr int KS = C::KS, KC = C::KC, AHEAD = C::AHEAD;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 15, g = lane >> 4;
  const int k0 = w.k0, k1 = w.k1, nc = (k1 - k0 + KC - 1) / KC;
  const uint16_t* xp[C::XP];
  u32x4 xr[C::XP], xo[KIND == HEADS ? C::XP : 1];  // (HEADS: the token's other feature)
  float c_own[C::XP], c_other[C::XP];
  long long other[C::XP];
  const bool mixed = KIND == HEADS && p.heads_mode != JK_HEADS_DECOUPLED;
  auto x_row = [&](int q) { return (tid + q * kThreads) / (KC / 8); };
  auto x_col = [&](int q) { return ((tid + q * kThreads) % (KC / 8)) * 8; };
  auto x_used = [&](int q) {
    return C::PIECES % kThreads == 0 || tid + q * kThreads < C::PIECES;
  };
#pragma unroll
  for (int q = 0; q < C::XP; ++q) {  // rows past the end repeat the last one; never stored
    int row = min(x_row(q), m - 1);
    if (KIND == PAIR) row = list[row] >> 1;
    if (KIND == DOWN) row = list[row];
    xp[q] = p.x + (long long)row * p.k;
    if constexpr (KIND == HEADS) {
      other[q] = (row & 1) ? -(long long)p.k : (long long)p.k;
      const float s_own = p.s_top[row], s_other = p.s_top[row ^ 1];
      c_own[q] = mixed && (row & 1) ? -p.alpha : s_own;
      c_other[q] = !mixed ? 0.f : (row & 1) ? p.beta : s_other;
    }
  }
  auto load_x = [&](int kc) {
#pragma unroll
    for (int q = 0; q < C::XP; ++q)
      if (x_used(q)) {
        const uint16_t* at = xp[q] + min(kc + x_col(q), k1 - 8);
        xr[q] = *reinterpret_cast<const u32x4*>(at);
        if constexpr (KIND == HEADS)
          if (mixed) xo[q] = *reinterpret_cast<const u32x4*>(at + other[q]);
      }
  };
  // (a term whose coefficient is zero is left out, so that a NaN in the other expert's feature cannot leak into a
  // decoupled head)
  auto mix = [&](u32x4 own, u32x4 oth, float c, float co) {
    u32x4 o;
    if constexpr (MT <= 2) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float lo = c != 0.f ? c * bf16_lo(own[j]) : 0.f, hi = c != 0.f ? c * bf16_hi(own[j]) : 0.f;
        if (mixed && co != 0.f) {
          lo += co * bf16_lo(oth[j]);
          hi += co * bf16_hi(oth[j]);
        }
        o[j] = bf16_bits_rne(lo) | (bf16_bits_rne(hi) << 16);
      }
    } else {  // (a third of the instructions, which count here; few rows wait for their weights, and are up to 1 % slower like this)
      const unsigned keep = c != 0.f ? ~0u : 0u, keep_other = co != 0.f ? ~0u : 0u;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float lo = c * bf16_lo(own[j] & keep), hi = c * bf16_hi(own[j] & keep);
        if (mixed) {
          lo += co * bf16_lo(oth[j] & keep_other);
          hi += co * bf16_hi(oth[j] & keep_other);
        }
        o[j] = dev::pack_bf16(lo, hi);
      }
    }
    return o;
  };
  auto park_x = [&](int buf) {
    if constexpr (KIND == HEADS) {
#pragma unroll
      for (int q = 0; q < C::XP; ++q) xr[q] = mix(xr[q], xo[q], c_own[q], c_other[q]);
    }
#pragma unroll
    for (int q = 0; q < C::XP; ++q)
      if (x_used(q)) *reinterpret_cast<u32x4*>(xbuf + buf * C::X_BYTES + x_row(q) * (C::LDX * 2) + x_col(q) * 2) = xr[q];
  };
  floatx4 acc[NF][MT];
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[f][t] = floatx4{0.f, 0.f, 0.f, 0.f};
  const unsigned char* x_lane = xbuf + r * (C::LDX * 2) + 16 * g;
  // k steps j0 .. j1 - 1 of chunk c, whose first k is kc; the following chunk, if there is one, starts at `next`.  X operands
  // are read LOOK products ahead of their use, and each weight register is asked for again once its last product is
  // issued.  The order is fixed step by step: left alone, the compiler puts each read right in front of its product
  // (90 rows of a draft layer's three products: 133 us, and 124 like this) and gathers the loads at the chunk's end.
  auto steps = [&](int c, int kc, int next, auto j0c, auto j1c, auto morec) {
    constexpr int J0 = decltype(j0c)::value, N = (decltype(j1c)::value - J0) * MT, LOOK = C::LOOK < N ? C::LOOK : N;
    const unsigned char* x = x_lane + (c & 1) * C::X_BYTES;
    bf16x8 b[LOOK + 1];
    auto read = [&](int i) { b[i % (LOOK + 1)] = *reinterpret_cast<const bf16x8*>(x + (i % MT) * 16 * (C::LDX * 2) + 64 * (J0 + i / MT)); };
#pragma unroll
    for (int i = 0; i < LOOK; ++i) read(i);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int j = J0 + i / MT, t = i % MT;
      if (i + LOOK < N) read(i + LOOK);
#pragma unroll
      for (int f = 0; f < NF; ++f) acc[f][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.a[f][j % AHEAD], b[i % (LOOK + 1)], acc[f][t], 0, 0, 0);
      if (t == MT - 1) {
        if (j + AHEAD < KS) w.load(kc + 32 * (j + AHEAD), j % AHEAD);
        else if (decltype(morec)::value) w.load(next + 32 * (j + AHEAD - KS), j % AHEAD);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  typedef std::integral_constant<int, 0> Zero;
  typedef std::integral_constant<int, KS < 4 ? KS : 4> Half;
  typedef std::integral_constant<int, KS> Whole;
  load_x(w.template chunk<KC>(0));
  park_x(0);
  __syncthreads();
  for (int c = 0; c + 1 < nc; ++c) {  // every chunk but the last is whole
    const int kn = w.template chunk<KC>(c + 1);
    load_x(kn);
    steps(c, w.template chunk<KC>(c), kn, Zero(), Whole(), std::true_type());
    park_x((c + 1) & 1);
    __syncthreads();
  }
  {
    const int c = nc - 1, kc = w.template chunk<KC>(c);
    steps(c, kc, 0, Zero(), Half(), std::false_type());
    if (KS > 4 && (k1 - k0) % KC == 0) steps(c, kc, 0, Half(), Whole(), std::false_type());
  }

  // A lane holds, for output row 16 t + r, columns (the wave's, 16 per fragment) + 4 g + (0..3): stored as it is, every
  // instruction would write 64 bytes of each of 16 rows (a 57 MB result of odd width: 41 us, and 18 like this).  So the rows are laid
  // out in LDS, as many as its X buffers hold at a time, and go out whole.
  constexpr int COLS = strip_rows(NF), LDO = COLS + 4, FIT = C::SMEM / (16 * LDO * 4), RT = FIT < MT ? FIT : MT;
  constexpr int OUT = KIND == PAIR ? COLS / 2 : COLS;  // output columns (PAIR: the gate's in front of the up projection's)
  static_assert(RT >= 1, "an output block fits");
  const bool vec = (p.n & 3) == 0 && (reinterpret_cast<size_t>(p.y) & 15) == 0 && (reinterpret_cast<size_t>(p.residual) & 7) == 0 &&
                   (reinterpret_cast<size_t>(p.out_bf16) & 7) == 0;
  float* tile = reinterpret_cast<float*>(xbuf);
  const int n0 = (int)blockIdx.x * OUT;
  auto y_row = [&](int row) { return (long long)(KIND == PAIR || KIND == DOWN ? list[row] : row); };
  // The statistics of a row's 128 columns, by half a wave with four columns a lane: the launch that read all logits again for them was 7 us of
  // 190 (20 rows, 128256 x 4096).  (With expf this was 0.7 us of every workgroup's end, and those of a CU come one after the other.)
  auto stats_of = [&](floatx4 v, int row, int col) {
    float top = -INFINITY, sum = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[e] = n0 + col + e < p.n ? v[e] : -INFINITY;
      top = fmaxf(top, v[e]);
    }
    top = dev::half_max(top);
    const float from = top > -INFINITY ? top : 0.f;  // (nothing sensible to subtract)
#pragma unroll
    for (int e = 0; e < 4; ++e) sum += dev::exp_scaled(v[e] - from, p.scale_hi, p.scale_lo);
    sum = dev::half_sum(sum);
    const int blocks = (p.n + kStatColumns - 1) / kStatColumns, at = (n0 + col) / kStatColumns;
    if ((lane & 31) == 0 && at < blocks) p.stats[(long long)row * blocks + at] = make_float2(top, sum);
  };
  // emit4 (emit1): element offset in the output, and where its four values (its value) are in LDS
  auto put = [&](auto emit4, auto emit1) {
#pragma unroll
    for (int t0 = 0; t0 < MT; t0 += RT) {
      if (16 * t0 >= m) break;
      __syncthreads();  // what was read here before has been used
#pragma unroll
      for (int t = t0; t < (t0 + RT < MT ? t0 + RT : MT); ++t)
#pragma unroll
        for (int f = 0; f < NF; ++f)
          *reinterpret_cast<floatx4*>(tile + (16 * (t - t0) + r) * LDO + wave * 16 * NF + 16 * f + 4 * g) = acc[f][t];
      __syncthreads();
      const int rows = min(16 * RT, m - 16 * t0);
      if (vec) {
#pragma unroll 4
        for (int i = tid; i < rows * (OUT / 4); i += kThreads) {
          const int row = i / (OUT / 4), col = i % (OUT / 4) * 4;
          if (n0 + col < p.n) emit4(y_row(16 * t0 + row) * p.n + n0 + col, reinterpret_cast<const floatx4*>(tile + row * LDO + col));
        }
      } else {
        for (int i = tid; i < rows * OUT; i += kThreads) {
          const int row = i / OUT, col = i % OUT;
          if (n0 + col < p.n) emit1(y_row(16 * t0 + row) * p.n + n0 + col, tile + row * LDO + col);
        }
      }
      if constexpr (KIND == HEADS)  // (half waves at a time: all lanes that a move between lanes asks take part)
        if (p.stats)
          for (int i = tid; i < rows * (OUT / 4); i += kThreads) {
            const int row = i / (OUT / 4), col = i % (OUT / 4) * 4;
            stats_of(*reinterpret_cast<const floatx4*>(tile + row * LDO + col), 16 * t0 + row, col);
          }
    }
  };
  const long long part = (long long)blockIdx.z * p.y_split;
  float* y = p.y + part;
  if constexpr (KIND == PAIR) {
    float* y2 = p.y2 + part;
    uint16_t* h = p.act;
    auto gated = [](float a, float b) { return a / (1.f + expf(-a)) * b; };
    if (p.act) {
      put(
          [&](long long at, const floatx4* v) {
            const floatx4 a = v[0], b = v[OUT / 4];
            uint2 o;
            o.x = bf16_bits_rne(gated(a[0], b[0])) | (bf16_bits_rne(gated(a[1], b[1])) << 16);
            o.y = bf16_bits_rne(gated(a[2], b[2])) | (bf16_bits_rne(gated(a[3], b[3])) << 16);
            *reinterpret_cast<uint2*>(h + at) = o;
          },
          [&](long long at, const float* v) { h[at] = (uint16_t)bf16_bits_rne(gated(v[0], v[OUT])); });
    } else {
      put(
          [&](long long at, const floatx4* v) {
            *reinterpret_cast<floatx4*>(y + at) = v[0];
            *reinterpret_cast<floatx4*>(y2 + at) = v[OUT / 4];
          },
          [&](long long at, const float* v) {
            y[at] = v[0];
            y2[at] = v[OUT];
          });
    }
  } else if (KIND == PLAIN && p.finish) {  // an undivided k range: the finished layer
    const uint16_t* res = p.residual;
    put(
        [&](long long at, const floatx4* pv) {
          floatx4 v = *pv;
          if (res) {
            const uint2 q = *reinterpret_cast<const uint2*>(res + at);
            v += floatx4{bf16_lo(q.x), bf16_hi(q.x), bf16_lo(q.y), bf16_hi(q.y)};
          }
          if (p.y) *reinterpret_cast<floatx4*>(p.y + at) = v;
          if (p.out_bf16) {
            uint2 o;
            o.x = bf16_bits_rne(v[0]) | (bf16_bits_rne(v[1]) << 16);
            o.y = bf16_bits_rne(v[2]) | (bf16_bits_rne(v[3]) << 16);
            *reinterpret_cast<uint2*>(p.out_bf16 + at) = o;
          }
        },
        [&](long long at, const float* pv) {
          float v = *pv;
          if (res) v += bf16_lo(res[at]);
          if (p.y) p.y[at] = v;
          if (p.out_bf16) p.out_bf16[at] = (uint16_t)bf16_bits_rne(v);
        });
  } else {
    // (parts of a split product are small and read again at once; whole results of tens of megabytes only push the
    // weights' way through the caches: 128256 x 4096, 80 rows: 253 us with ordinary stores, 242 with these)
    const bool parts = p.ksplit > 1;
    put(
        [&](long long at, const floatx4* v) {
          if (parts) *reinterpret_cast<floatx4*>(y + at) = *v;
          else __builtin_nontemporal_store(*v, reinterpret_cast<floatx4*>(y + at));
        },
        [&](long long at, const float* v) { y[at] = *v; });
  }
}

// The leading arguments are in scalar registers when a wave starts (a compiler option for this file, fourteen words at most): the
// others take 0.3 us to come from memory, and the first requests for weights wait for none of them.  (With those of ring_gemm.hip, us,
// in memory / so: experts, 8 rows, eight of 512 x 512 15.0 / 14.2, 64 rows, four of 1024 x 2048 29.6 / 28.4.)
template <int MT, int NF, Kind KIND>
__global__ __launch_bounds__(kThreads, 2) void stream_gemm_kernel(const uint16_t* lead_w, const uint16_t* lead_w2, long long w_batch, int n, int k,
                                                                  int ksplit, int strips, const uint16_t* x, int rows, StreamGemmArgs p) {
  p.w = lead_w;
  p.w2 = lead_w2;
  p.w_batch = w_batch;
  p.n = n;
  p.k = k;
  p.ksplit = ksplit;
  p.x = x;
  p.m = rows;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, e = blockIdx.y;
  // (PAIR: four waves have gate rows, four the same rows of the up projection; with both in one wave, two fragments of
  // half as many k steps each, the short pieces of a row cost 5 - 9 % of the bandwidth unless rows are a power of two long)
  const int n_base = KIND == PAIR ? ((int)blockIdx.x * 4 + (wave & 3)) * 16 * NF : ((int)blockIdx.x * 8 + wave) * 16 * NF;
  Weights<NF, KIND> w;
  w.start(p, strips, n_base, e, wave, lane & 15, lane >> 4);
  // (an expert's chunks have the same order whatever its number of rows, at most 128: KC is 256 in all of those variants)
  constexpr int KC = Cfg<MT, NF>::KC;
  const int first = w.template chunk<KC>(0);
#pragma unroll
  for (int j = 0; j < steps_ahead(NF); ++j) w.load(first + 32 * j, j);
  if constexpr (KIND == PLAIN || KIND == HEADS) {
    strip_products<MT, NF, KIND>(p, w, p.m, nullptr, smem, e);
  } else {
    // The rows that chose expert e, in order.  Every wave makes the whole list (the same one) for itself: its LDS
    // operations complete in order, so no barrier is needed before it reads its own entries.
    int* list = reinterpret_cast<int*>(smem);
    int m = 0;
    for (int i0 = 0; i0 < p.m; i0 += 64) {
      const int row = i0 + lane;
      const bool mine = row < p.m && (p.sel[2 * row] == e || p.sel[2 * row + 1] == e);
      const unsigned long long v = __ballot(mine);
      if (mine) list[m + __popcll(v & ((1ull << lane) - 1ull))] = 2 * row + (p.sel[2 * row] == e ? 0 : 1);
      m += __popcll(v);
    }
    if (m == 0) return;  // nobody chose it (the whole workgroup: nobody waits at a later barrier)
    unsigned char* xbuf = smem + kListBytes;
    if constexpr (MT <= 2) {
      strip_products<MT, NF, KIND>(p, w, m, list, xbuf, e);
    } else {
      // The loop for just as many 16-row blocks as there are: conditions inside one loop for the most keep its loads and
      // products apart (75 rows, two experts of 4992 x 11136: 223 us for the call, 194 like this).
      auto run = [&](auto t) {
        constexpr int T = decltype(t)::value;
        if constexpr (T <= MT) strip_products<T, NF, KIND>(p, w, m, list, xbuf, e);
      };
      switch ((m + 15) / 16) {
        case 1:
        case 2: run(std::integral_constant<int, 2>()); break;
        case 3: run(std::integral_constant<int, 3>()); break;
        case 4: run(std::integral_constant<int, 4>()); break;
        case 5: run(std::integral_constant<int, 5>()); break;
        case 6: run(std::integral_constant<int, 6>()); break;
        default: run(std::integral_constant<int, 8>()); break;
      }
    }
  }
}

template <int MT, int NF, Kind KIND>
hipError_t launch(const StreamGemmArgs& p, hipStream_t stream) {
  static LdsLimitRaised raised;
  // (more than half of the LDS: one workgroup per CU.  Two of them fit a CU's registers with few rows, and are put there
  // while other CUs have none: 1 row, two of 5 experts of 5632 x 12928: 280 us for the call, 215 like this)
  constexpr int need = Cfg<MT, NF>::SMEM + (KIND == PLAIN || KIND == HEADS ? 0 : kListBytes), smem = need > 82 * 1024 ? need : 82 * 1024;
  if (hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(stream_gemm_kernel<MT, NF, KIND>), smem, raised); e != hipSuccess)
    return e;
  constexpr int COLS = strip_rows(NF) / (KIND == PAIR ? 2 : 1);
  const int strips = (p.n + COLS - 1) / COLS;
  return launch_kernel(stream_gemm_kernel<MT, NF, KIND>, dim3((unsigned)strips, (unsigned)p.batch, (unsigned)p.ksplit), dim3(kThreads), smem, stream,
                     p.w, p.w2, p.w_batch, p.n, p.k, p.ksplit, strips, p.x, p.m, p);
}

}  // namespace

// Parts of the k range.  A CU draws at most about 31 bytes per ns, all of them together 5 750 (their HBM share): a turn
// of fewer workgroups than CUs takes as long as its workgroups alone.  A part more costs its fp32 partial results,
// written and read once at about 4 000 bytes per ns, and the first one what `split_ns` says (another launch).  The count
// with the least time by this estimate (in ns), fewer parts where it is a tie; a part keeps at least 128 of k.
// `batch`: products in one launch that really run.  *ns (or null): the estimate.
int stream_gemm_ksplit(int m, int n, int k, int batch, bool pair, int split_ns, double* ns) {
  const int cus = device_cu_count();
  const double rows = strip_rows(m <= 128 ? 1 : 2), out = (double)n * (pair ? 2 : 1);
  const int units = k / 128, top = units < 64 ? units : 64;
  double best_t = 0.0;
  int best = 1;
  for (int s = 1; s <= top; ++s) {
    const double bytes = 2.0 * rows * 128.0 * ((units + s - 1) / s), alone = bytes / 31.0;
    const long long all = (long long)std::ceil(out / rows) * batch * s, full = all / cus, rest = all % cus;
    auto turn = [&](double wgs) { return 1500.0 + (alone > bytes * wgs / 5750.0 ? alone : bytes * wgs / 5750.0); };
    const double parts_t = s > 1 ? split_ns + 2.0 * 4.0 * s * m * out * batch / 4000.0 : 0.0;
    const double t = (double)full * turn(cus) + (rest ? turn((double)rest) : 0.0) + parts_t;
    if (s == 1 || t < 0.98 * best_t) {
      best_t = t;
      best = s;
    }
  }
  if (ns) *ns = best_t;
  return best;
}

namespace {
// Columns of a strip / 128 where a workgroup has the whole k range.  Wide strips start less often (about 2 us a turn of
// workgroups), narrow ones fill the last turn better.  (m = 112, 127835 x 1408: 115 us in strips of 128, 104 in strips of
// 256; 142, 74527 x 5888: 335 and 265 in strips of 256 and 384; 80, 128256 x 4096: 204 and 207 in strips of 128 and 256.)
// More than 128 rows leave no LDS for strips of 128, more than 160 no registers for strips of 384.
int strip_width(int n, int k, int narrowest, int widest) {
  double best_t = 0.0;
  int best = narrowest;
  for (int nf = narrowest; nf <= widest; ++nf) {
    const int strips = (n + 128 * nf - 1) / (128 * nf), turns = (strips + device_cu_count() - 1) / device_cu_count();
    const double cu_t = turns * 2.0 * k * 128.0 * nf / 31.0, hbm_t = 2.0 * n * k / 5750.0;
    const double t = (cu_t > hbm_t ? cu_t : hbm_t) + 2000.0 * turns;
    if (nf == narrowest || t < 0.97 * best_t) {
      best_t = t;
      best = nf;
    }
  }
  return best;
}

template <int MT, Kind KIND = PLAIN>
hipError_t launch_plain(const StreamGemmArgs& p, hipStream_t stream) {
  if constexpr (MT <= 8) {
    return p.ksplit == 1 && strip_width(p.n, p.k, 1, 2) == 2 ? launch<MT, 2, KIND>(p, stream) : launch<MT, 1, KIND>(p, stream);
  } else if constexpr (MT <= 10) {
    return p.ksplit == 1 && strip_width(p.n, p.k, 2, 3) == 3 ? launch<MT, 3, PLAIN>(p, stream) : launch<MT, 2, PLAIN>(p, stream);
  } else {
    return launch<MT, 2, PLAIN>(p, stream);
  }
}
}  // namespace

// Every workgroup mixes the rows for itself instead of a launch in front of it (5 us, of which 2.5 show).  All kernels, us,
// with the launch / without: 2 rows of 32000 x 4096 57.7 / 55.0, 20 rows 59.7 / 57.1, 128256 x 4096 197.7 / 195.8; the whole
// call, 40 rows of 32000 x 4096 64.0 / 62.3, 48 of 12159 x 5632 47.9 / 44.2, 64 of 128256 x 4096 232.3 / 225.6, with both
// features in a row 232.5 / 231.4; 128 of 128256 x 4096 291 / 307 and 290 / 328: so up to four row blocks of 16.
hipError_t launch_stream_gemm_heads(const StreamGemmArgs& p, hipStream_t stream) {
  switch ((p.m + 15) / 16) {
    case 1: return launch_plain<1, HEADS>(p, stream);
    case 2: return launch_plain<2, HEADS>(p, stream);
    case 3: return launch_plain<3, HEADS>(p, stream);
    case 4: return launch_plain<4, HEADS>(p, stream);
    default: return hipErrorInvalidValue;
  }
}
hipError_t launch_stream_gemm(const StreamGemmArgs& p, hipStream_t stream) {
  switch ((p.m + 15) / 16) {
    case 1: return launch_plain<1>(p, stream);
    case 2: return launch_plain<2>(p, stream);
    case 3: return launch_plain<3>(p, stream);
    case 4: return launch_plain<4>(p, stream);
    case 5: return launch_plain<5>(p, stream);
    case 6: return launch_plain<6>(p, stream);
    case 7:
    case 8: return launch_plain<8>(p, stream);
    case 9:
    case 10: return launch_plain<10>(p, stream);
    case 11:
    case 12: return launch_plain<12>(p, stream);
    case 13: case 14: case 15:
    case 16: return launch_plain<16>(p, stream);
    default: return hipErrorInvalidValue;
  }
}
namespace {
// (an expert may have been chosen by every row)
template <Kind KIND>
hipError_t launch_experts(const StreamGemmArgs& p, hipStream_t stream) {
  switch ((p.m + 15) / 16) {
    case 1: return launch<1, 1, KIND>(p, stream);
    case 2: return launch<2, 1, KIND>(p, stream);
    case 3:
    case 4: return launch<4, 1, KIND>(p, stream);
    case 5:
    case 6: return launch<6, 1, KIND>(p, stream);
    case 7:
    case 8: return launch<8, 1, KIND>(p, stream);
    default: return hipErrorInvalidValue;
  }
}
}  // namespace

hipError_t launch_stream_gemm_pair(const StreamGemmArgs& p, hipStream_t stream) { return launch_experts<PAIR>(p, stream); }
hipError_t launch_stream_gemm_down(const StreamGemmArgs& p, hipStream_t stream) { return launch_experts<DOWN>(p, stream); }

// ------------------------------------------------------------------ few output columns, few rows
namespace {
// What the products' first requests are made of stands in front as arguments of its own, in scalar registers when a wave starts (see
// stream_gemm_kernel): the operands, their sizes, a workgroup's rows of W (strip, one of `strips`) and of X, parts of the k range
// and places in a row of the grid.  The rest is for the end.
struct NarrowArgs {
  const uint16_t* residual;
  float* y;
  uint16_t* out_bf16;
  float* part;             // parts > 1: their sums, one workgroup's behind the other's
  unsigned long long* words;  // and a word per strip and block, kWordStep apart
  unsigned long long tag;
};
struct NarrowCall {
  const uint16_t *x, *w;
  int m, n, k, strip, strips, rows, parts;
  NarrowArgs end;
};
// Y = X . W^T (+ residual) for up to 128 rows and at most 64 columns per CU: a workgroup per CU has its strip of weight rows and
// all of k, its waves every eighth (fourth) 64 of k each (128-byte lines of W's and X's rows), and adds the waves' sums up
// in LDS.  Against parts of k per workgroup it saves writing the partial results and the launch that adds them up; in exchange
// every CU draws all of X from its L2.  What bounds it is HBM's share of the weights and, beyond some twenty rows, what a CU
// draws: 51 bytes per ns straight into LDS (global_load_lds_dwordx4), 47 through registers, 38 where neighbouring lanes do not
// ask for neighbouring addresses, as in the matrix operands' layout, whoever else draws.  So both operands come by LDS, each
// wave's through a ring of its own, up to six units ahead: no barriers, no registers.  With many rows and a long k two
// workgroups share a strip of twice the rows: half of X for each, and the second of them to finish adds up both (1.3 us:
// four parts save no more than their meeting costs).  Many rows of few columns are shared instead: two workgroups have a strip
// of twice the width and half of X's rows each and go through k in step, so that one of them draws the strip's weights from the
// L2 that both share (each with a start of its own 80 x 8192 x 8192 took 47 us, and takes 35).
// Measured (us, weights cold, before / now; before: weights in the operands' layout, X through registers, or strips of 128
// rows in parts of k and a second launch): 4096 x 4096, 8 rows 8.0 / 7.9, 16 8.9 / 8.3, 40 12.3 / 10.9, 64 15.0 / 12.1; 6144 x
// 4096, 8 11.1 / 10.7, 40 15.3 / 13.5, 64 18.2 / 15.9; 4096 x 8192, 8 14.4 / 14.1, 40 21.3 / 17.4, 64 22.9 / 20.0; 12288 x
// 4096, 45 26.9 / 21.3; 8192 x 16384, 20 60.0 / 48.6.  With X's rows shared: 4096 x 4096, 64 rows 12.5 / 11.9, 80 18.3 / 13.0, 128
// 21.3 / 15.8; 1024 x 2048, 64 6.2 / 5.2, 80 10.3 / 6.1; 3072 x 1024, 128 16.9 / 6.5; 8192 x 4096, 80 23.7 / 19.8.  Reading the weights alone takes 7.0, 9.5, 12.3, ..., 43.
// RG: groups of eight rows of X; NF: groups of 16 weight rows

// waves of a workgroup: eight, or four where LDS has no room for two units of each
constexpr int narrow_waves(int groups, int frags) { return 2 * 8 * (2 * frags + groups) <= 158 ? 8 : 4; }
constexpr int kWordStep = 32;  // (256 bytes: an atomic takes 11 ns of the memory channel that has its word)

// A wave's units of W and X, UK of k each, on their way through its own part of LDS: rows of 128 bytes, their 16-byte chunks
// in an order that spreads the matrix operands' reads over the banks
template <int RG, int NF, int WAVES>
struct NarrowCfg {
  static constexpr int UK = 64;
  static constexpr int MT = (RG + 1) / 2, TILES = NF * MT;
  static constexpr int ROW = 2 * UK, CHUNKS = ROW / 16, RPI = 8;  // bytes and chunks of a row, rows of a transfer
  static constexpr int WI = 2 * NF, XI = RG, PER = WI + XI;  // transfers of a unit
  static constexpr int FIT = 158 / (WAVES * PER), DEPTH = FIT < 6 ? FIT : 6;  // units in flight
  static constexpr int RING = DEPTH * PER * 1024;  // bytes of a wave
  static constexpr int SUMS = WAVES * TILES * 1024;
  static constexpr int SMEM = WAVES * RING + 1024 > SUMS ? WAVES * RING + 1024 : SUMS;  // (the rows that the last of 16 lack)
  static_assert(DEPTH >= 2, "LDS plan");
  static __device__ __forceinline__ int swizzle(int row) { return row & 7; }
};

template <int RG, int NF, int WAVES>
__global__ __launch_bounds__(64 * WAVES, WAVES / 4) void narrow_gemm_kernel(const uint16_t* w, const uint16_t* x, int m_all, int n, int k,
                                                                            int strip_len, int strips, int rows, int parts, int places,
                                                                            NarrowArgs p) {
  using C = NarrowCfg<RG, NF, WAVES>;
  constexpr int MT = C::MT, TILES = C::TILES, UK = C::UK, STEPS = UK / 32;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  floatx4* sums = reinterpret_cast<floatx4*>(smem);  // [wave][tile][lane], behind the loop
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), r = lane & 15, g = lane >> 4;
  const int blk = blockIdx.x, id = xcd_place(blk, places);  // (neighbours on one XCD share lines of Y)
  // (the blocks of X's rows are the grid's second dimension: what shares a strip's weights runs on one XCD, and in step)
  const int halves = parts - 1, strip = id >> halves;  // (one or two parts)
  if (strip >= strips) return;  // (the whole workgroup, see xcd_grid)
  const int z = id - (strip << halves), row0 = (int)blockIdx.y * rows, m = min(m_all - row0, rows);
  const int meet = strip + (int)blockIdx.y * strips;
  const int n_base = strip * strip_len, n_end = min(n_base + strip_len, n);
  const int units = (int)((unsigned)k / (unsigned)UK), u0 = (z * units) >> halves, u1 = ((z + 1) * units) >> halves;
  // (byte offsets from one scalar address each; rows past the end repeat the last one, and are not stored)
  const uint16_t *w0 = dev::uniform_ptr(w + (long long)n_base * k), *x0 = dev::uniform_ptr(x + (long long)row0 * k);
  const int lrow = lane / C::CHUNKS, lcol = 16 * (lane % C::CHUNKS ^ C::swizzle(lrow));
  unsigned wr[C::WI], xr[C::XI];
#pragma unroll
  for (int i = 0; i < C::WI; ++i) wr[i] = (unsigned)min(C::RPI * i + lrow, n_end - 1 - n_base) * (unsigned)k * 2u + lcol;
#pragma unroll
  for (int i = 0; i < C::XI; ++i) xr[i] = (unsigned)min(C::RPI * i + lrow, m - 1) * (unsigned)k * 2u + lcol;
  unsigned char* ring = smem + wave * C::RING;
  const unsigned ring_at = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)ring;
  const int count = (u1 - u0 - wave + WAVES - 1) / WAVES;  // this wave's units
  // (workgroups start at different units, see Weights::chunk: in 32nds of the wave's, five from XCD to XCD and one from each workgroup to the
  // next there.  A remainder by the number of units, 5 blk + blk / 8, was 20 instructions in front of the first request, us, so / like
  // this: 45 x 12288 x 4096 21.6 / 20.7, 80 x 8192 x 8192 35.1 / 33.9, 40 x 4096 x 8192 17.3 / 16.4, with the leading arguments in registers)
  const int rot = count > 0 ? (int)__umulhi((unsigned)(5 * (blk & 7) + (blk >> 3)) << 27, (unsigned)count) : 0;
  auto ask = [&](int j, int slot) {
    const int u = j + rot, at = (u0 + wave + WAVES * (u < count ? u : u - count)) * UK;
    const unsigned to = ring_at + slot * (C::PER * 1024);
#pragma unroll
    for (int i = 0; i < C::WI; ++i) dev::dma16(w0 + at, wr[i], to + 1024 * i);
#pragma unroll
    for (int i = 0; i < C::XI; ++i) dev::dma16(x0 + at, xr[i], to + 1024 * (C::WI + i));
  };
  // (four waves: two sums each, so that none is of more products than with eight)
  constexpr int SETS = 8 / WAVES;
  static_assert(SETS == 1 || SETS == STEPS, "a set per step");
  floatx4 acc[SETS][NF][MT];
#pragma unroll
  for (int q = 0; q < SETS; ++q)
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
      for (int t = 0; t < MT; ++t) acc[q][f][t] = floatx4{0.f, 0.f, 0.f, 0.f};
  int at[STEPS];  // of a lane's chunk of a row
#pragma unroll
  for (int s = 0; s < STEPS; ++s) at[s] = r * C::ROW + 16 * ((4 * s + g) ^ C::swizzle(r));
  bf16x8 a[NF][STEPS], b[MT][STEPS];
  auto take = [&](int slot) {  // (and the slot may be filled again)
    const unsigned char* from = ring + slot * (C::PER * 1024);
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
#pragma unroll
      for (int f = 0; f < NF; ++f) a[f][s] = *reinterpret_cast<const bf16x8*>(from + f * 16 * C::ROW + at[s]);
#pragma unroll
      for (int t = 0; t < MT; ++t) b[t][s] = *reinterpret_cast<const bf16x8*>(from + C::WI * 1024 + t * 16 * C::ROW + at[s]);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  };
  auto multiply = [&] {
#pragma unroll
    for (int s = 0; s < STEPS; ++s)
#pragma unroll
      for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int f = 0; f < NF; ++f) {
          floatx4& sum = acc[s % SETS][f][t];
          sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[f][s], b[t][s], sum, 0, 0, 0);
        }
  };
#pragma unroll
  for (int j = 0; j < C::DEPTH; ++j)
    if (j < count) ask(j, j);
  int j = 0, slot = 0;
  for (; j + C::DEPTH < count; ++j) {
    dev::wait_vm<(C::DEPTH - 1) * C::PER>();
    take(slot);
    ask(j + C::DEPTH, slot);
    multiply();
    slot = slot + 1 == C::DEPTH ? 0 : slot + 1;
  }
  // (count - j units are on their way, at most DEPTH)
  auto rest = [&](auto self, auto leftc) -> void {
    constexpr int LEFT = decltype(leftc)::value;
    if constexpr (LEFT > 0) {
      if (count - j >= LEFT) {
        dev::wait_vm<(LEFT - 1) * C::PER>();
        take(slot);
        multiply();
        slot = slot + 1 == C::DEPTH ? 0 : slot + 1;
        ++j;
      }
      self(self, std::integral_constant<int, LEFT - 1>());
    }
  };
  rest(rest, std::integral_constant<int, C::DEPTH>());
  __syncthreads();  // (the sums take the place of the ring)
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      floatx4 v = acc[0][f][t];
      if constexpr (SETS == 2) v += acc[1][f][t];
      sums[(wave * TILES + f * MT + t) * 64 + lane] = v;
    }
  __syncthreads();
  const bool vec = (n & 3) == 0 && (reinterpret_cast<size_t>(p.y) & 15) == 0 && (reinterpret_cast<size_t>(p.residual) & 7) == 0 &&
                   (reinterpret_cast<size_t>(p.out_bf16) & 7) == 0;
  auto finish = [&](int i, floatx4 v) {
    // (a lane of a tile has row lane % 16 of X and four consecutive columns)
    const int tile = i >> 6, row = (tile % MT) * 16 + (i & 15), col = n_base + (tile / MT) * 16 + ((i & 63) >> 4) * 4;
    if (row >= m || col >= n_end) return;
    const long long at = (long long)(row0 + row) * n + col;
    if (vec && col + 4 <= n_end) {
      if (p.residual) {
        const uint2 q = *reinterpret_cast<const uint2*>(p.residual + at);
        v += floatx4{bf16_lo(q.x), bf16_hi(q.x), bf16_lo(q.y), bf16_hi(q.y)};
      }
      if (p.y) *reinterpret_cast<floatx4*>(p.y + at) = v;
      if (p.out_bf16) {
        uint2 o;
        o.x = bf16_bits_rne(v[0]) | (bf16_bits_rne(v[1]) << 16);
        o.y = bf16_bits_rne(v[2]) | (bf16_bits_rne(v[3]) << 16);
        *reinterpret_cast<uint2*>(p.out_bf16 + at) = o;
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (col + e >= n_end) break;
        float s = v[e];
        if (p.residual) s += bf16_lo(p.residual[at + e]);
        if (p.y) p.y[at + e] = s;
        if (p.out_bf16) p.out_bf16[at + e] = (uint16_t)bf16_bits_rne(s);
      }
    }
  };
  constexpr int QUADS = TILES * 64;  // of a workgroup's results
  float* own_part = p.part + (size_t)(meet * parts + z) * (QUADS * 4);
  for (int i = tid; i < QUADS; i += 64 * WAVES) {
    floatx4 part[WAVES];
#pragma unroll
    for (int w = 0; w < WAVES; ++w) part[w] = sums[w * QUADS + i];
#pragma unroll
    for (int d = 1; d < WAVES; d *= 2)  // (two and two: fewer roundings on the way of each)
#pragma unroll
      for (int w = 0; w < WAVES; w += 2 * d) part[w] += part[w + d];
    if (parts == 1) finish(i, part[0]);
    else dev::store_through(own_part + 4 * i, __builtin_bit_cast(dev::store_u32x4, part[0]));
  }
  if (parts == 1) return;
  if (!dev::second_to_meet(p.words + (size_t)meet * kWordStep, p.tag, reinterpret_cast<int*>(smem))) return;
  const auto both = __builtin_amdgcn_make_buffer_rsrc(p.part + (size_t)meet * (2 * QUADS * 4), 0, 2 * QUADS * 16, 0x00020000);
  for (int i = tid; i < QUADS; i += 64 * WAVES) {  // (the same sum whoever comes second)
    const u32x4 low = __builtin_amdgcn_raw_buffer_load_b128(both, i * 16, 0, dev::kDeviceScope);
    const u32x4 high = __builtin_amdgcn_raw_buffer_load_b128(both, i * 16, QUADS * 16, dev::kDeviceScope);
    finish(i, __builtin_bit_cast(floatx4, low) + __builtin_bit_cast(floatx4, high));
  }
}

template <int RG, int NF>
hipError_t launch_narrow(const NarrowCall& p, int blocks, hipStream_t stream) {
  static LdsLimitRaised raised;
  constexpr int WAVES = narrow_waves(RG, NF);
  constexpr int smem = NarrowCfg<RG, NF, WAVES>::SMEM;
  if (hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(narrow_gemm_kernel<RG, NF, WAVES>), smem, raised); e != hipSuccess) return e;
  // (Where the row blocks of a strip ran on different XCDs, with 121 strips of 56, 80 x 6760 x 7296 took 40.7 us, and takes 36.9.)
  const dim3 grid((unsigned)xcd_grid(p.strips * p.parts, blocks), (unsigned)blocks);
  return launch_kernel(narrow_gemm_kernel<RG, NF, WAVES>, grid, dim3(64 * WAVES), smem, stream, p.w, p.x, p.m, p.n, p.k, p.strip, p.strips, p.rows,
                     p.parts, (int)grid.x, p.end);
}
template <int RG>
hipError_t launch_narrow_rows(const NarrowCall& p, int blocks, hipStream_t stream) {
  switch ((p.strip + 15) / 16) {
    case 1: return launch_narrow<RG, 1>(p, blocks, stream);
    case 2: return launch_narrow<RG, 2>(p, blocks, stream);
    case 3: return launch_narrow<RG, 3>(p, blocks, stream);
    case 4: return launch_narrow<RG, 4>(p, blocks, stream);
    default: return hipErrorInvalidValue;
  }
}
}  // namespace

// Strips of at most 64 weight rows, X's rows in blocks of at most 64, and k in one or two parts, by the estimated time: HBM's
// share of the weights beside what a CU draws of its weights and of X, a start and an end, the meeting of two parts, and four
// waves instead of eight.  Over 45 shapes (1 - 64 rows, 832 - 16384 columns, k 768 - 16384) the estimate is off by 4 % and the choice 0.4 %
// behind the better.
NarrowPlan narrow_plan(int m, int n, int k) {
  const int cus = device_cu_count();
  NarrowPlan best{0, 0, 0, 0, 0, 0.0};
  for (int blocks = (m + 63) / 64; blocks <= 2; ++blocks) {
    const int rows = ((m + blocks - 1) / blocks + 7) / 8 * 8;
    if (rows * (blocks - 1) >= m) break;  // (nothing left for the last one)
    for (int parts = 1; parts <= 2; ++parts) {
      const int most = cus / (parts * blocks);  // strips
      if (most < 1 || n > 64 * (long long)most) break;
      const int strip = ((n + most - 1) / most + 3) / 4 * 4, frags = (strip + 15) / 16;
      const double cu = 2.0 * k / parts * (strip + rows) / 65.0, hbm = 2.0 * n * k / 6400.0;
      const double ns = 2700.0 + std::cbrt(cu * cu * cu + hbm * hbm * hbm) + (parts > 1 ? 1250.0 : 0.0) + (narrow_waves(rows / 8, frags) == 4 ? 1350.0 : 0.0);
      if (best.parts == 0 || ns < best.ns) best = NarrowPlan{strip, (n + strip - 1) / strip, rows, blocks, parts, ns};
    }
  }
  return best;
}
size_t narrow_gemm_bytes(const NarrowPlan& plan) {
  if (plan.parts <= 1) return 0;
  const size_t tiles = (size_t)((plan.strip + 15) / 16) * ((plan.rows + 15) / 16);
  return (size_t)plan.strips * plan.blocks * (kWordStep * 8 + plan.parts * tiles * 1024);
}
hipError_t launch_narrow_gemm(const StreamGemmArgs& g, const NarrowPlan& plan, void* workspace, hipStream_t stream) {
  NarrowCall p;
  p.x = g.x; p.w = g.w;
  p.m = g.m; p.n = g.n; p.k = g.k;
  p.strip = plan.strip; p.strips = plan.strips; p.rows = plan.rows; p.parts = plan.parts;
  p.end.residual = g.residual; p.end.y = g.y; p.end.out_bf16 = g.out_bf16;
  p.end.words = static_cast<unsigned long long*>(workspace);
  p.end.part = reinterpret_cast<float*>(static_cast<char*>(workspace) + (size_t)plan.strips * plan.blocks * (kWordStep * 8));
  p.end.tag = meeting_tag();
  switch (plan.rows / 8) {
    case 1: return launch_narrow_rows<1>(p, plan.blocks, stream);
    case 2: return launch_narrow_rows<2>(p, plan.blocks, stream);
    case 3: return launch_narrow_rows<3>(p, plan.blocks, stream);
    case 4: return launch_narrow_rows<4>(p, plan.blocks, stream);
    case 5: return launch_narrow_rows<5>(p, plan.blocks, stream);
    case 6: return launch_narrow_rows<6>(p, plan.blocks, stream);
    case 7: return launch_narrow_rows<7>(p, plan.blocks, stream);
    case 8: return launch_narrow_rows<8>(p, plan.blocks, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace jk
