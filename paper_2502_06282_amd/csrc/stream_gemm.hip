// Products of few rows with weight matrices of tens to hundreds of megabytes (gfx950): the draft layer's linear layers,
// its experts' projections, and output heads over a small vocabulary.  Y[M, N] = X[M, K] . W[N, K]^T, M <= 256, bf16
// operands, fp32 accumulation.
//
// What bounds it: the weight stream, and for a few tens of megabytes the round trip to memory in front of it.  So a wave
// fetches its weights straight into registers in MFMA layout (v_mfma_f32_16x16x32_bf16: 16 rows of 64 bytes per
// instruction, the other half of each 128-byte line with the next k step), 8 KB of them in flight from the first
// cycle on, each register asked for again as soon as its product is issued; only X goes through LDS, one chunk of k
// ahead of its use, shared by the workgroup's eight waves; one barrier per chunk.  Narrow strips (128 weight rows) and
// whole k ranges where that gives every CU a workgroup, k split into as many parts as it takes otherwise.
// Measured on an MI355X (weights cold, 40 rows, us): 4096 x 8192 15.2, 6144 x 4096 13.5, 4096 x 4096 9.4, 1024 x 2048
// 4.9; 16 x 4096 x 4096 98, 8 x 4096 x 4096 49 (5.5 TB/s; a plain read of a gigabyte runs at 5.75).  The kernel that
// these calls used before (skinny_gemm_kernel: weights through LDS rings, strips of 512 rows, at most eight k parts)
// took 35.3, 22.9, 21.3, 15.2, 114 and 61 us.  It is still the better one for very many weight rows (128256 x 4096,
// 20 rows: 177 us against 180), where a workgroup per CU has a strip of 512 to itself.  Non-temporal loads (-10 %) and
// chunks of 512 (no difference) were tried.
#include "jk_internal.h"

namespace jk {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 512;  // 8 waves

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
enum Kind { PLAIN, PAIR, DOWN };

template <int MT, int KC, Kind KIND>
struct Cfg {
  static constexpr int NF = KIND == PAIR || MT > 8 ? 2 : 1;  // 16-row weight fragments per wave
  static constexpr int COLS = KIND == PAIR ? 128 : 128 * NF;  // output columns per workgroup
  static constexpr int KS = KC / 32;                          // MFMA k steps per chunk
  static constexpr int LDX = KC + 8;  // bf16 per LDS row: 16 bytes of padding spread the rows over the banks
  static constexpr int PIECES = MT * 16 * (KC / 8);           // 16-byte pieces of an X chunk
  static constexpr int XP = (PIECES + kThreads - 1) / kThreads;
  static constexpr int X_BYTES = MT * 16 * LDX * 2;
  static constexpr int LIST = KIND == PLAIN ? 0 : 512;        // the rows that chose this expert (at most 128)
  static constexpr int SMEM = LIST + 2 * X_BYTES;
  static_assert(SMEM <= 160 * 1024, "LDS plan");
  // operand reads of X run one k step ahead of the products; with many rows there are no registers for that, and
  // the two waves of a SIMD cover each other's reads instead
  static constexpr int NB = MT <= 8 ? 2 : 1;
};

template <int MT, int KC, Kind KIND>
__global__ __launch_bounds__(kThreads, 2) void stream_gemm_kernel(StreamGemmArgs p) {
  using C = Cfg<MT, KC, KIND>;
  constexpr int NF = C::NF, KS = C::KS, NB = C::NB;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 15, g = lane >> 4;
  const int e = blockIdx.y;
  int* list = reinterpret_cast<int*>(smem);
  int m = p.m;
  if (KIND != PLAIN) {
    // The rows that chose expert e, in order.  Every wave makes the whole list (the same one) for itself: its LDS
    // operations complete in order, so no barrier is needed before it reads its own entries.
    m = 0;
    for (int i0 = 0; i0 < p.m; i0 += 64) {
      const int row = i0 + lane;
      const bool mine = row < p.m && (p.sel[2 * row] == e || p.sel[2 * row + 1] == e);
      const unsigned long long v = __ballot(mine);
      if (mine) list[m + __popcll(v & ((1ull << lane) - 1ull))] = row;
      m += __popcll(v);
    }
    if (m == 0) return;  // nobody chose it (the whole workgroup: nobody waits at a later barrier)
  }
  const int nt = KIND == PLAIN ? MT : (m + 15) / 16;  // 16-row blocks of X in use
  const uint16_t* px = p.x + (long long)e * p.x_batch;
  const uint16_t* pw = p.w + (long long)e * p.w_batch;
  const int n_base = (int)blockIdx.x * C::COLS + wave * (C::COLS / 8);
  // this part's k range, in units of 128 (whole chunks but perhaps for the last one of the range)
  const int units = p.k / 128;
  const int k0 = (int)((long long)blockIdx.z * units / p.ksplit) * 128, k1 = (int)((long long)(blockIdx.z + 1) * units / p.ksplit) * 128;
  const int nc = (k1 - k0 + KC - 1) / KC;
  // Workgroups start at different chunks and wrap around: rows often lie a power of two apart, so that workgroups in
  // step would all ask the same few memory channels (16 x 4096 x 4096: 115 us in step, 98 us like this; 32000 x 4096:
  // 58 and 46).  Workgroups run on the eight XCDs in turn, so the start has to vary within every eighth of them too.
  // (A half chunk at the end stays last.)
  const int whole = (k1 - k0) / KC;
  const unsigned wg = blockIdx.x + gridDim.x * blockIdx.y;
  const int rot = whole > 0 ? (int)((5u * wg + (wg >> 3)) % (unsigned)whole) : 0;
  auto chunk_k = [&](int c) {
    const int t = c + rot;
    return k0 + (c < whole ? (t < whole ? t : t - whole) : c) * KC;
  };

  const uint16_t* wp[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    const int row = min(n_base + (KIND == PAIR ? 0 : 16 * f) + r, p.n - 1);  // rows past the end repeat the last one; never stored
    const uint16_t* base = KIND == PAIR && f == 1 ? p.w2 + (long long)e * p.w_batch : pw;
    wp[f] = base + (long long)row * p.k + 8 * g;
  }
  bf16x8 a[NF][KS];
  // (what lies past a half chunk at the end of the range is fetched from inside it and not used)
  auto load_w = [&](int kc, int j) {
    const int k = min(kc + 32 * j, k1 - 32);
#pragma unroll
    for (int f = 0; f < NF; ++f) a[f][j] = *reinterpret_cast<const bf16x8*>(wp[f] + k);
  };
#pragma unroll
  for (int j = 0; j < KS; ++j) load_w(chunk_k(0), j);

  const uint16_t* xp[C::XP];
  u32x4 xr[C::XP];
  auto x_row = [&](int q) { return (tid + q * kThreads) / (KC / 8); };
  auto x_col = [&](int q) { return ((tid + q * kThreads) % (KC / 8)) * 8; };
  auto x_used = [&](int q) {
    return KIND == PLAIN ? (C::PIECES % kThreads == 0 || tid + q * kThreads < C::PIECES) : x_row(q) < 16 * nt;
  };
#pragma unroll
  for (int q = 0; q < C::XP; ++q) {  // rows past the end repeat the last one; never stored
    int row = min(x_row(q), m - 1);
    if (KIND == PAIR) row = list[row];
    xp[q] = px + (long long)row * p.k;
  }
  auto load_x = [&](int kc) {
#pragma unroll
    for (int q = 0; q < C::XP; ++q)
      if (x_used(q)) xr[q] = *reinterpret_cast<const u32x4*>(xp[q] + min(kc + x_col(q), k1 - 8));
  };
  auto park_x = [&](int buf) {
#pragma unroll
    for (int q = 0; q < C::XP; ++q)
      if (x_used(q)) *reinterpret_cast<u32x4*>(smem + C::LIST + buf * C::X_BYTES + x_row(q) * (C::LDX * 2) + x_col(q) * 2) = xr[q];
  };
  floatx4 acc[NF][MT];
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[f][t] = floatx4{0.f, 0.f, 0.f, 0.f};
  bf16x8 b[NB][MT];
  const unsigned char* x_lane = smem + C::LIST + r * (C::LDX * 2) + 16 * g;
  auto read_x = [&](int c, int j) {
#pragma unroll
    for (int t = 0; t < MT; ++t)
      if (KIND == PLAIN || t < nt)
        b[j % NB][t] = *reinterpret_cast<const bf16x8*>(x_lane + (c & 1) * C::X_BYTES + t * 16 * (C::LDX * 2) + 64 * j);
  };
  auto products = [&](int j) {
#pragma unroll
    for (int t = 0; t < MT; ++t)
      if (KIND == PLAIN || t < nt) {
#pragma unroll
        for (int f = 0; f < NF; ++f) acc[f][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[f][j], b[j % NB][t], acc[f][t], 0, 0, 0);
      }
  };
  load_x(chunk_k(0));
  park_x(0);
  __syncthreads();
  for (int c = 0; c + 1 < nc; ++c) {  // every chunk but the last is whole
    const int kn = chunk_k(c + 1);
    load_x(kn);
    if (NB == 2) read_x(c, 0);
#pragma unroll
    for (int j = 0; j < KS; ++j) {
      if (NB == 1 || j + 1 < KS) read_x(c, NB == 1 ? j : j + 1);
      products(j);
      load_w(kn, j);
      // (left alone, the compiler gathers all loads at the chunk's end, with nothing in flight by then)
      asm volatile("" ::: "memory");
    }
    park_x((c + 1) & 1);
    __syncthreads();
  }
  {
    const int c = nc - 1;
    auto last = [&](int j0, int j1) {
      if (NB == 2) read_x(c, j0);
#pragma unroll
      for (int j = j0; j < j1; ++j) {
        if (NB == 1 || j + 1 < j1) read_x(c, NB == 1 ? j : j + 1);
        products(j);
      }
    };
    last(0, 4);
    if (KS > 4 && (k1 - k0) % KC == 0) last(4, KS);
  }

  // lane (r, g) holds, for output row 16 t + r, columns block + 4 g + (0..3)
  const bool vec = (p.n & 3) == 0 && (reinterpret_cast<size_t>(p.y) & 15) == 0 && (reinterpret_cast<size_t>(p.residual) & 7) == 0 &&
                   (reinterpret_cast<size_t>(p.out_bf16) & 7) == 0;
  if (KIND == PAIR && p.act) {
    uint16_t* h = p.act + (long long)e * p.act_batch;
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      const int row = 16 * t + r, n = n_base + 4 * g;
      if (row >= m || n >= p.n) continue;
      float o[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = acc[0][t][i] / (1.f + expf(-acc[0][t][i])) * acc[NF - 1][t][i];
      uint2 v;
      v.x = bf16_bits_rne(o[0]) | (bf16_bits_rne(o[1]) << 16);
      v.y = bf16_bits_rne(o[2]) | (bf16_bits_rne(o[3]) << 16);
      *reinterpret_cast<uint2*>(h + (long long)row * p.n + n) = v;  // (n is a multiple of 128)
    }
    return;
  }
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    float* y = (KIND == PAIR && f == 1 ? p.y2 : p.y) + (long long)e * p.y_batch + (long long)blockIdx.z * p.y_split;
    const int n = n_base + (KIND == PAIR ? 0 : 16 * f) + 4 * g;
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      const int row = 16 * t + r;
      if (row >= m) continue;
      const long long at = (long long)row * p.n + n;
      if (KIND == PLAIN && p.finish) {  // an undivided k range: the finished layer
        const uint16_t* res = p.residual;
        if (vec && n < p.n) {
          floatx4 v = acc[f][t];
          if (res) {
            const uint2 q = *reinterpret_cast<const uint2*>(res + at);
            v += floatx4{bf16_lo(q.x), bf16_hi(q.x), bf16_lo(q.y), bf16_hi(q.y)};
          }
          if (p.y) *reinterpret_cast<floatx4*>(y + at) = v;
          if (p.out_bf16) {
            uint2 o;
            o.x = bf16_bits_rne(v[0]) | (bf16_bits_rne(v[1]) << 16);
            o.y = bf16_bits_rne(v[2]) | (bf16_bits_rne(v[3]) << 16);
            *reinterpret_cast<uint2*>(p.out_bf16 + at) = o;
          }
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (n + i < p.n) {
              float v = acc[f][t][i];
              if (res) v += bf16_lo(res[at + i]);
              if (p.y) y[at + i] = v;
              if (p.out_bf16) p.out_bf16[at + i] = (uint16_t)bf16_bits_rne(v);
            }
        }
      } else if (vec && n < p.n) {
        *reinterpret_cast<floatx4*>(y + at) = acc[f][t];
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (n + i < p.n) y[at + i] = acc[f][t][i];
      }
    }
  }
}

template <int MT, int KC, Kind KIND>
hipError_t launch(const StreamGemmArgs& p, hipStream_t stream) {
  using C = Cfg<MT, KC, KIND>;
  static LdsLimitRaised raised;
  if (hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(stream_gemm_kernel<MT, KC, KIND>), C::SMEM, raised); e != hipSuccess)
    return e;
  hipLaunchKernelGGL((stream_gemm_kernel<MT, KC, KIND>), dim3((unsigned)((p.n + C::COLS - 1) / C::COLS), (unsigned)p.batch, (unsigned)p.ksplit),
                     dim3(kThreads), C::SMEM, stream, p);
  return hipGetLastError();
}

}  // namespace

// Parts of the k range.  A CU draws at most about 31 bytes per ns, all of them together 5 750 (their HBM share); a part
// more costs its fp32 partial results, written and read once at about 4 000 bytes per ns.  The count with the least
// time by this estimate (in ns), fewer parts where it is a tie; a part keeps at least 128 of k.  `batch`: products in
// one launch that really run.
int stream_gemm_ksplit(int m, int n, int k, int batch, bool pair) {
  const int cus = device_cu_count();
  const int cols = pair || m <= 128 ? 128 : 256;
  const double strips = (double)((n + cols - 1) / cols) * batch;
  const double weights = 2.0 * n * k * batch * (pair ? 2 : 1);
  const int units = k / 128, top = units < 64 ? units : 64;
  double best_t = 0.0;
  int best = 1;
  for (int s = 1; s <= top; ++s) {
    const double part_k = 128.0 * ((units + s - 1) / s);
    const double turns = (double)(((long long)strips * s + cus - 1) / cus);
    const double cu_t = turns * 2.0 * cols * (pair ? 2 : 1) * part_k / 31.0, hbm_t = weights / 5750.0;
    const double parts_t = s > 1 ? 2.0 * 4.0 * s * m * (double)n * batch * (pair ? 2 : 1) / 4000.0 : 0.0;
    const double t = (cu_t > hbm_t ? cu_t : hbm_t) + parts_t;
    if (s == 1 || t < 0.98 * best_t) {
      best_t = t;
      best = s;
    }
  }
  return best;
}

hipError_t launch_stream_gemm(const StreamGemmArgs& p, hipStream_t stream) {
  switch ((p.m + 15) / 16) {
    case 1: return launch<1, 256, PLAIN>(p, stream);
    case 2: return launch<2, 256, PLAIN>(p, stream);
    case 3: return launch<3, 256, PLAIN>(p, stream);
    case 4: return launch<4, 256, PLAIN>(p, stream);
    case 5: return launch<5, 256, PLAIN>(p, stream);
    case 6: return launch<6, 256, PLAIN>(p, stream);
    case 7:
    case 8: return launch<8, 256, PLAIN>(p, stream);
    case 9:
    case 10: return launch<10, 128, PLAIN>(p, stream);
    case 11:
    case 12: return launch<12, 128, PLAIN>(p, stream);
    case 13: case 14: case 15:
    case 16: return launch<16, 128, PLAIN>(p, stream);
    default: return hipErrorInvalidValue;
  }
}
hipError_t launch_stream_gemm_pair(const StreamGemmArgs& p, hipStream_t stream) {
  switch ((p.m + 15) / 16) {
    case 1: return launch<1, 256, PAIR>(p, stream);
    case 2: return launch<2, 256, PAIR>(p, stream);
    case 3: return launch<3, 256, PAIR>(p, stream);
    case 4: return launch<4, 256, PAIR>(p, stream);
    case 5:
    case 6: return launch<6, 256, PAIR>(p, stream);
    case 7:
    case 8: return launch<8, 128, PAIR>(p, stream);
    default: return hipErrorInvalidValue;
  }
}
hipError_t launch_stream_gemm_down(const StreamGemmArgs& p, hipStream_t stream) {
  switch ((p.m + 15) / 16) {
    case 1: return launch<1, 256, DOWN>(p, stream);
    case 2: return launch<2, 256, DOWN>(p, stream);
    case 3: return launch<3, 256, DOWN>(p, stream);
    case 4: return launch<4, 256, DOWN>(p, stream);
    case 5:
    case 6: return launch<6, 256, DOWN>(p, stream);
    case 7:
    case 8: return launch<8, 256, DOWN>(p, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace jk
