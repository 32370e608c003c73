// Token acceptance over the verified draft tree (gfx950).
//
// Section 2.1 of the paper: candidates are judged in order with acceptance
// probability min(1, p/q); at a rejection the distribution becomes
// norm(max(0, p - q)) (steps 2-3).  Section 3.2: greedy decoding is strict
// top-1 verification.  On a tree the rule is applied sibling by sibling, left
// to right (Section 3.1.2 puts the higher-scoring expert's candidates on the
// left), each node carrying its own draft distribution.
//
// Kernels
//   greedy_kernel       greedy calls: rows reduced and trees walked in one launch
//   row_reduce_kernel   one pass over the [rows, vocab] logits: per (row,
//                       chunk) either (max, argmax) or (max, sum exp) partials
//   walk_greedy_kernel  (calls without a workspace, or of more trees than the
//                       workspace has words) one workgroup per tree: merges the partials per row,
//                       marks every node whose token equals its parent row's
//                       argmax, then descends from the prefix
//   walk_sample_kernel  one workgroup per tree: descends from the prefix; a
//                       rejection costs one pass over the vocabulary that
//                       writes the unnormalised residual to the workspace and
//                       reduces its sum; the bonus token is found by a blocked
//                       prefix sum over the final distribution.  All sampling
//                       arithmetic is fp64: the inverse-CDF draw resolves steps
//                       of ~1/vocab, which fp32 terms cannot do reproducibly
#include <cstdlib>
#include <mutex>

#include "jk_device.h"
#include "jk_internal.h"
#include "jk_wave.h"
#include "walk_alone.h"

namespace jk {
namespace {

constexpr int kChunk = 4096;        // vocabulary entries per row_reduce workgroup
constexpr int kWalkThreads = 1024;  // threads of a sampling walk

__host__ __device__ inline int n_chunks(int vocab) { return (vocab + kChunk - 1) / kChunk; }

// ------------------------------------------------------------------ row reductions
template <bool SAMPLE>
__global__ __launch_bounds__(256) void row_reduce_kernel(const float* __restrict__ logits, int vocab,
                                                         double temp, float* __restrict__ pmax,
                                                         int* __restrict__ pidx, double* __restrict__ psum) {
  __shared__ float s_max[4];
  __shared__ int s_idx[4];
  __shared__ double s_sum[4];
  const int chunk = blockIdx.x;
  const long long row = blockIdx.y;
  const float* src = logits + row * vocab;
  const int v0 = chunk * kChunk;
  const int v1 = min(vocab, v0 + kChunk);
  const int tid = threadIdx.x;

  float vals[16];
  float best = -INFINITY;
  int bidx = 0x7fffffff;
  const bool vec = ((vocab & 3) == 0);  // rows stay 16-byte aligned
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int v = v0 + (j * 256 + tid) * 4;
    if (vec && v + 3 < v1) {
      const float4 x = *reinterpret_cast<const float4*>(src + v);
      vals[4 * j] = x.x; vals[4 * j + 1] = x.y; vals[4 * j + 2] = x.z; vals[4 * j + 3] = x.w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) vals[4 * j + e] = (v + e < v1) ? src[v + e] : -INFINITY;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float x = vals[4 * j + e];
      if (x > best) { best = x; bidx = v + e; }  // ascending v inside a thread keeps the lowest id
    }
  }
  // block (max, lowest index of the max)
  for (int o = 32; o > 0; o >>= 1) {
    const float ob = __shfl_xor(best, o);
    const int oi = __shfl_xor(bidx, o);
    if (ob > best || (ob == best && oi < bidx)) { best = ob; bidx = oi; }
  }
  if ((tid & 63) == 0) { s_max[tid >> 6] = best; s_idx[tid >> 6] = bidx; }
  __syncthreads();
  best = s_max[0]; bidx = s_idx[0];
#pragma unroll
  for (int w = 1; w < 4; ++w)
    if (s_max[w] > best || (s_max[w] == best && s_idx[w] < bidx)) { best = s_max[w]; bidx = s_idx[w]; }

  const long long slot = row * gridDim.x + chunk;
  if (!SAMPLE) {
    if (tid == 0) { pmax[slot] = best; pidx[slot] = bidx; }
    return;
  }
  // sum of exp(x/T - max/T) over the chunk, all in fp64 (same operations as the definition,
  // so a decision of the walk differs from exact arithmetic only at ~1e-15 relative)
  const double mref = (best == -INFINITY) ? 0.0 : (double)best / temp;
  double acc = 0.0;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc += exp((double)vals[i] / temp - mref);
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
  if ((tid & 63) == 0) s_sum[tid >> 6] = acc;
  __syncthreads();
  if (tid == 0) { pmax[slot] = best; psum[slot] = s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3]; }
}

using dev::report;
using dev::sanitize_parent;

// ------------------------------------------------------------------ greedy walk
__global__ __launch_bounds__(128) void walk_greedy_kernel(int n_tree, int nch, int vocab, int max_depth,
                                                          const int* __restrict__ tokens,
                                                          const int* __restrict__ parent,
                                                          const float* __restrict__ pmax,
                                                          const int* __restrict__ pidx, int* __restrict__ out_path,
                                                          int* __restrict__ out_len, int* __restrict__ out_bonus,
                                                          unsigned* err) {
  __shared__ int amax[JK_MAX_TREE + 1];
  __shared__ int par_s[JK_MAX_TREE];
  __shared__ int ok[JK_MAX_TREE];
  const int b = blockIdx.x, tid = threadIdx.x;
  const int rows = n_tree + 1;
  for (int r = tid; r < rows; r += blockDim.x) {
    const long long base = ((long long)b * rows + r) * nch;
    float best = -INFINITY;
    int bi = 0x7fffffff;
    for (int c0 = 0; c0 < nch; c0 += 8) {  // eight partials in flight at a time
      float v[8];
      int id[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const bool in = c0 + u < nch;
        v[u] = in ? pmax[base + c0 + u] : -INFINITY;
        id[u] = in ? pidx[base + c0 + u] : 0x7fffffff;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)  // chunks ascend in token id: strict > keeps the lowest id
        if (v[u] > best) { best = v[u]; bi = id[u]; }
    }
    amax[r] = (bi == 0x7fffffff) ? 0 : bi;  // a row of -inf only: id 0, the first maximum
  }
  if (tid < n_tree) par_s[tid] = sanitize_parent(parent[(long long)b * n_tree + tid], tid, err);
  __syncthreads();
  if (tid < n_tree) {
    const int tk = tokens[(long long)b * n_tree + tid];
    const int tc = min(max(tk, 0), vocab - 1);  // as in the sampling walks: an id outside the vocabulary is clamped, and reported
    if (tc != tk) report(err, kDevErrBadToken);
    ok[tid] = (tc == amax[par_s[tid] + 1]);
  }
  __syncthreads();
  if (tid < 64) {  // wave 0 descends: the first accepted child of c, found with two ballots per level
    const int lane = tid;
    const bool in0 = lane < n_tree, in1 = lane + 64 < n_tree;
    const int p0 = in0 ? par_s[lane] : -2, p1 = in1 ? par_s[lane + 64] : -2;
    const bool ok0 = in0 && ok[lane], ok1 = in1 && ok[lane + 64];
    int c = -1, len = 0;
    // (nodes are numbered topologically: a child has a larger index than its parent; the walk
    // stops at max_depth accepted nodes, and the extra token then comes from the last one's row)
    while (len < max_depth) {
      const unsigned long long m0 = __ballot(ok0 && p0 == c), m1 = __ballot(ok1 && p1 == c);
      const int k = m0 ? __ffsll((long long)m0) - 1 : (m1 ? 63 + __ffsll((long long)m1) : -1);
      if (k < 0) break;
      if (lane == 0) out_path[(long long)b * max_depth + len] = k;
      ++len;
      c = k;
    }
    if (lane != 0) return;
    for (int i = len; i < max_depth; ++i) out_path[(long long)b * max_depth + i] = -1;
    out_len[b] = len;
    out_bonus[b] = amax[c + 1];
  }
}

// ------------------------------------------------------------------ greedy walk in one launch
constexpr int kGreedyLoads = 8;  // 16 bytes a load, at most so many of them per thread, all in flight
constexpr int greedy_chunk(int threads) { return threads * kGreedyLoads * 4; }  // most vocabulary entries per workgroup

// (What the first requests are made of stands in front as arguments of its own, in scalar registers when a wave starts: a compiler
// option for this file, fourteen words at most.  The others take 0.3 us to come from memory: four trees of 60 nodes, 32000 entries
// 8.84 us with all of them in memory, 8.65 like this.)
struct GreedyParams {
  int max_depth;
  uint64_t* part;   // [rows][chunks] (bits of the maximum, its lowest index)
  unsigned* words;  // the header's lines; see greedy_word (jk_words.h)
  int *out_path, *out_len, *out_bonus;
  unsigned* err;
};

// The rows' maxima and the walk in one kernel: a workgroup per (chunk, row) leaves its (max, argmax) in memory and counts
// itself; the one that finds itself the last of its tree walks it.  Nobody waits, so it does not matter how many run at
// once.  What bounds it is the stream of logits behind a launch, a reduction and three trips to memory (result, counter,
// results back); a second launch for the walk cost more than the last two.  Measured (us, two launches / one): four trees of
// 60 nodes, 32000 entries 10.5 / 8.9 (31 MB); one tree 7.4 / 5.7; one tree, 128256 entries 12.2 / 9.4; 20 nodes 6.1 / 4.8;
// 64 trees 90 / 88.  The workgroups of a tree run on different XCDs, whose L2s know nothing of each other: results go through to memory
// and are on their way back before the counter moves, and are read past the caches (device scope).
template <int THREADS, int LOADS>
__global__ __launch_bounds__(THREADS) void greedy_kernel(const float* logits, int vocab, int chunk, unsigned mg_rows, int n_tree, const int* parent,
                                                         const int* tokens, int nch, int all_rows, GreedyParams p) {
  constexpr int kWaves = THREADS / 64;
  __shared__ float s_max[kWaves];
  __shared__ int s_idx[kWaves];
  __shared__ int amax[JK_MAX_TREE + 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int rows = n_tree + 1;
  const int row = blockIdx.y, b = (int)__umulhi((unsigned)row, mg_rows);
  const float* src = logits + (long long)row * vocab;
  const int v0 = (int)blockIdx.x * chunk, v1 = min(vocab, v0 + chunk);
  const bool vec = (vocab & 3) == 0;  // rows stay 16-byte aligned
  float4 x[LOADS];
#pragma unroll
  for (int j = 0; j < LOADS; ++j) {
    const int v = v0 + (j * THREADS + tid) * 4;
    x[j] = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
    if (vec) {
      if (v < v1) x[j] = *reinterpret_cast<const float4*>(src + v);  // (chunks are multiples of four)
    } else {
      if (v < v1) x[j].x = src[v];
      if (v + 1 < v1) x[j].y = src[v + 1];
      if (v + 2 < v1) x[j].z = src[v + 2];
      if (v + 3 < v1) x[j].w = src[v + 3];
    }
  }
  // (what the walk needs besides, on its way as well: only the first wave walks, nodes lane and lane + 64)
  const int n0 = min(lane, n_tree - 1), n1 = min(lane + 64, n_tree - 1);
  int pa0 = 0, pa1 = 0, tk0 = 0, tk1 = 0;
  if (wave == 0) {
    const long long base = (long long)b * n_tree;
    pa0 = parent[base + n0]; pa1 = parent[base + n1];
    tk0 = tokens[base + n0]; tk1 = tokens[base + n1];
  }
  float best = -INFINITY;
  int bidx = 0x7fffffff;
#pragma unroll
  for (int j = 0; j < LOADS; ++j) {  // ascending inside a thread: strict > keeps the lowest id
    const int v = v0 + (j * THREADS + tid) * 4;
    if (x[j].x > best) { best = x[j].x; bidx = v; }
    if (x[j].y > best) { best = x[j].y; bidx = v + 1; }
    if (x[j].z > best) { best = x[j].z; bidx = v + 2; }
    if (x[j].w > best) { best = x[j].w; bidx = v + 3; }
  }
  const float wmax = dev::wave_max(best);
  const int widx = dev::wave_min(best == wmax ? bidx : 0x7fffffff);
  if (lane == 0) { s_max[wave] = wmax; s_idx[wave] = widx; }
  __syncthreads();
  if (wave != 0) return;
  best = lane < kWaves ? s_max[lane] : -INFINITY;
  bidx = lane < kWaves ? s_idx[lane] : 0x7fffffff;
  const float bmax = dev::wave_max(best);
  const int bmin = dev::wave_min(best == bmax ? bidx : 0x7fffffff);
  // first among the parts of the row, then, the row's last one, among the rows of the tree (words: the trees', then the rows')
  bool last = true;
  if (lane == 0) {
    dev::store_through(p.part + (size_t)row * nch + blockIdx.x, dev::store_u32x2{__float_as_uint(bmax), (unsigned)bmin});
    dev::wait_vm<0>();
    auto arrive = [&](int i, int of) {
      unsigned* word = greedy_word(p.words, i);
      if (of > 1 && __hip_atomic_fetch_add(word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != (unsigned)of - 1) return false;
      if (of > 1) __hip_atomic_store(word, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return true;
    };
    last = arrive((int)__umulhi((unsigned)all_rows, mg_rows) + row, nch) && arrive(b, rows);
  }
  if (!__builtin_amdgcn_readfirstlane((int)last)) return;

  // ---- the tree's last workgroup: everybody's results are in memory
  for (int r = lane; r < rows; r += 64) {
    const uint64_t* part = p.part + ((size_t)b * rows + r) * nch;
    float m = -INFINITY;
    int id = 0x7fffffff;
    for (int c0 = 0; c0 < nch; c0 += 8) {  // eight partials in flight at a time
      uint64_t w[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) w[u] = __hip_atomic_load(part + min(c0 + u, nch - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
      for (int u = 0; u < 8; ++u)  // chunks ascend in token id: strict > keeps the lowest id (the last one again changes nothing)
        if (__uint_as_float((unsigned)w[u]) > m) { m = __uint_as_float((unsigned)w[u]); id = (int)(w[u] >> 32); }
    }
    amax[r] = id == 0x7fffffff ? 0 : id;  // a row of -inf only: id 0, the first maximum
  }
  auto checked = [&](int k, int& pa, int& tk) {
    if (k >= n_tree) { pa = -2; return; }
    pa = sanitize_parent(pa, k, p.err);
    const int tc = min(max(tk, 0), vocab - 1);  // an id outside the vocabulary is clamped, and reported
    if (tc != tk) report(p.err, kDevErrBadToken);
    tk = tc;
  };
  checked(lane, pa0, tk0);
  checked(lane + 64, pa1, tk1);
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // (one wave: its LDS operations complete in order)
  const bool ok0 = pa0 > -2 && tk0 == amax[max(pa0, -1) + 1], ok1 = pa1 > -2 && tk1 == amax[max(pa1, -1) + 1];
  int c = -1, len = 0;
  // (nodes are numbered topologically: a child has a larger index than its parent; the walk stops at max_depth accepted
  // nodes, and the extra token then comes from the last one's row)
  while (len < p.max_depth) {
    const unsigned long long m0 = __ballot(ok0 && pa0 == c), m1 = __ballot(ok1 && pa1 == c);
    const int k = m0 ? __ffsll((long long)m0) - 1 : (m1 ? 63 + __ffsll((long long)m1) : -1);
    if (k < 0) break;
    if (lane == 0) p.out_path[(long long)b * p.max_depth + len] = k;
    ++len;
    c = k;
  }
  for (int i = len + lane; i < p.max_depth; i += 64) p.out_path[(long long)b * p.max_depth + i] = -1;
  if (lane == 0) {
    p.out_len[b] = len;
    p.out_bonus[b] = amax[c + 1];
  }
}

template <int THREADS>
hipError_t launch_greedy(const AcceptArgs& a, const GreedyParams& p, int chunk, int parts, hipStream_t stream) {
  const int rows = a.batch * (a.n_tree + 1), loads = (chunk + THREADS * 4 - 1) / (THREADS * 4);
  const unsigned mg_rows = (unsigned)((1ull << 32) / (unsigned)(a.n_tree + 1) + 1);  // (rows of a tree: at least two)
  auto launch = [&](auto kernel) {
    return launch_kernel(kernel, dim3(parts, rows), dim3(THREADS), 0, stream, a.logits, a.vocab, chunk, mg_rows, a.n_tree, a.parent, a.tokens, parts,
                         rows, p);
  };
  if (loads <= 1) return launch(greedy_kernel<THREADS, 1>);
  if (loads <= 2) return launch(greedy_kernel<THREADS, 2>);
  return loads <= 4 ? launch(greedy_kernel<THREADS, 4>) : launch(greedy_kernel<THREADS, kGreedyLoads>);
}

// ------------------------------------------------------------------ sampling walk
struct WalkParams {
  dev::AloneParams walk;
  int nch;
  const float* pmax;
  const double* psum;
};

__global__ __launch_bounds__(kWalkThreads) void walk_sample_kernel(WalkParams p) {
  __shared__ dev::AloneShared<kWalkThreads> sh;
  const int b = blockIdx.x;
  dev::walk_alone<kWalkThreads>(p.walk, b, sh, [&](int r, double& row_max, double& row_z) {
    const long long base = ((long long)b * (p.walk.n_tree + 1) + r) * p.nch;
    float mx = -INFINITY;
    for (int i = 0; i < p.nch; ++i) mx = fmaxf(mx, p.pmax[base + i]);
    const double mref = (mx == -INFINITY) ? 0.0 : (double)mx / p.walk.temp;
    double z = 0.0;
    for (int i = 0; i < p.nch; ++i) {
      const float mc = p.pmax[base + i];
      if (mc != -INFINITY) z += p.psum[base + i] * exp((double)mc / p.walk.temp - mref);
    }
    row_max = mref;
    row_z = z;
  });
}

// ------------------------------------------------------------------ library-owned scratch
// For the entry point that takes no workspace (callers that cannot allocate device memory):
// the (max, argmax) partials of the greedy walk live in this array instead.  Every GPU the
// library runs on holds its own copy at its own address until the process ends; in host code
// the array's name is only a handle for hipGetSymbolAddress, never a device address.
static __device__ __align__(256) unsigned char scratch[JK_STATIC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices];  // device address of `scratch` on each device, looked up once

hipError_t scratch_address(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));  // the current device's copy
    if (e != hipSuccess) return e;
    if (!ptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

// Where do consecutive workgroups run?  Every workgroup of a small grid records the id of the XCD
// it is on (the attention kernel merges its key splits inside one XCD's L2 and relies on the
// hardware dealing workgroup n to XCD n mod 8).
__global__ void xcd_probe_kernel(unsigned* out) {
  unsigned id;
  asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(id));
  if (threadIdx.x == 0) out[blockIdx.x] = id & 0xfu;
}

struct WsLayout {
  size_t words, coop, pmax, pidx, psum, resid, total;  // (the error word's header sits in front of them)
};
WsLayout ws_layout(int batch, int n_tree, int vocab, int mode, bool caller_workspace = true) {
  WsLayout w{};
  const size_t rows = (size_t)batch * (n_tree + 1);
  const size_t slots = rows * n_chunks(vocab);
  auto up = [](size_t x) { return (x + 255) / 256 * 256; };
  size_t off = kWsErrBytes;
  // the per-tree blocks of the cooperative walk come first, in every caller's workspace and for
  // every mode: their words keep their place and are never overlaid by another call's partials,
  // so a workspace needs zeroing only once whatever calls take turns on it (the library's own
  // scratch array serves greedy calls only and has no such blocks)
  // (greedy calls count in words that attention calls use too and leave at zero, at their place in an attention workspace)
  w.words = off; off = caller_workspace ? kAttnHeaderBytes : off;
  w.coop = off; off += caller_workspace ? up(accept_coop_bytes()) : 0;
  w.pmax = off; off += up(slots * sizeof(float));
  w.pidx = off; off += up(slots * sizeof(int));
  w.psum = off; off += (mode == JK_SAMPLE) ? up(slots * sizeof(double)) : 0;
  w.resid = off; off += (mode == JK_SAMPLE) ? up((size_t)batch * 2 * vocab * sizeof(double)) : 0;
  w.total = off;
  return w;
}

}  // namespace

size_t accept_workspace_bytes(int batch, int n_tree, int vocab, int mode) {
  return ws_layout(batch, n_tree, vocab, mode).total;
}

// Synchronous, for jk_init: resolves the scratch array of the current device and runs the probe
// in it.  *round_robin: workgroups whose numbers agree modulo 8 were all on one XCD.
hipError_t probe_xcd_placement(hipStream_t stream, bool* round_robin) {
  constexpr int kProbeWgs = 256;
  void* base = nullptr;
  hipError_t e = scratch_address(&base);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(xcd_probe_kernel, dim3(kProbeWgs), dim3(64), 0, stream, static_cast<unsigned*>(base));
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  unsigned ids[kProbeWgs];
  e = hipMemcpyAsync(ids, base, sizeof(ids), hipMemcpyDeviceToHost, stream);
  if (e != hipSuccess) return e;
  e = hipStreamSynchronize(stream);
  if (e != hipSuccess) return e;
  bool ok = true;
  for (int n = 8; n < kProbeWgs; ++n) ok = ok && ids[n] == ids[n & 7];
  *round_robin = ok;
  return hipSuccess;
}

size_t accept_greedy_static_bytes(int batch, int n_tree, int vocab) {
  return ws_layout(batch, n_tree, vocab, JK_GREEDY, false).total;
}

// Greedy acceptance with the partials in the library's own scratch array: no workspace argument, nothing allocated, and the
// two kernels that launch_accept has for calls without counting words (the scratch array has none that are known to be
// zero, as the one launch needs them).  Nothing in the array needs clearing: every partial the walk reads is written by the
// reduction of the same call.
hipError_t launch_accept_greedy_static(const AcceptArgs& a, hipStream_t stream) {
  void* base = nullptr;
  hipError_t e = scratch_address(&base);
  if (e != hipSuccess) return e;
  const WsLayout w = ws_layout(a.batch, a.n_tree, a.vocab, JK_GREEDY, false);
  if (w.total > (size_t)JK_STATIC_SCRATCH_BYTES) return hipErrorInvalidValue;  // (checked by the caller too)
  char* ws = static_cast<char*>(base);
  float* pmax = reinterpret_cast<float*>(ws + w.pmax);
  int* pidx = reinterpret_cast<int*>(ws + w.pidx);
  const int nch = n_chunks(a.vocab);
  hipLaunchKernelGGL(row_reduce_kernel<false>, dim3(nch, a.batch * (a.n_tree + 1)), dim3(256), 0, stream, a.logits,
                     a.vocab, 1.0, pmax, pidx, static_cast<double*>(nullptr));
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(walk_greedy_kernel, dim3(a.batch), dim3(128), 0, stream, a.n_tree, nch, a.vocab, a.max_depth, a.tokens,
                     a.parent, pmax, pidx, a.out_path, a.out_len, a.out_bonus, static_cast<unsigned*>(nullptr));
  return hipGetLastError();
}

hipError_t launch_accept(const AcceptArgs& a, hipStream_t stream) {
  const WsLayout w = ws_layout(a.batch, a.n_tree, a.vocab, a.mode);
  char* ws = static_cast<char*>(a.workspace);
  float* pmax = reinterpret_cast<float*>(ws + w.pmax);
  int* pidx = reinterpret_cast<int*>(ws + w.pidx);
  double* psum = reinterpret_cast<double*>(ws + w.psum);
  double* resid = reinterpret_cast<double*>(ws + w.resid);
  const int nch = n_chunks(a.vocab);
  const dim3 grid(nch, a.batch * (a.n_tree + 1));
  const int rows = a.batch * (a.n_tree + 1);
  if (a.mode == JK_GREEDY && a.batch + rows <= kGreedyWords) {
    // A workgroup for each CU at least, in chunks no smaller than the two launches'.  Workgroups of 1024 threads where all of
    // them are resident at once, else of 512 (us, 512 / 1024 threads: four trees of 60 nodes, 32000 entries 9.3 / 8.9, eight
    // 16.3 / 15.3; five, 50257 entries 20.6 / 22.4; four of 100 nodes, 128256 entries 40.7 / 43.1).
    const int cus = device_cu_count();
    int threads = 1024, parts = (a.vocab + greedy_chunk(threads) - 1) / greedy_chunk(threads);
    if ((long long)parts * rows > 2 * cus) {  // (more than are resident at once)
      threads = 512;
      parts = (a.vocab + greedy_chunk(threads) - 1) / greedy_chunk(threads);
    }
    if (parts < cus / rows) parts = cus / rows < nch ? cus / rows : nch;
    GreedyParams gp;
    gp.max_depth = a.max_depth;
    const int chunk = ((a.vocab + parts - 1) / parts + 3) / 4 * 4;
    gp.part = reinterpret_cast<uint64_t*>(ws + w.pmax);
    gp.words = reinterpret_cast<unsigned*>(ws + w.words);
    gp.out_path = a.out_path; gp.out_len = a.out_len; gp.out_bonus = a.out_bonus;
    gp.err = reinterpret_cast<unsigned*>(ws);
    return threads == 1024 ? launch_greedy<1024>(a, gp, chunk, parts, stream) : launch_greedy<512>(a, gp, chunk, parts, stream);
  }
  if (a.mode == JK_GREEDY) {
    hipLaunchKernelGGL(row_reduce_kernel<false>, grid, dim3(256), 0, stream, a.logits, a.vocab, 1.0, pmax, pidx,
                       psum);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(walk_greedy_kernel, dim3(a.batch), dim3(128), 0, stream, a.n_tree, nch, a.vocab, a.max_depth,
                       a.tokens, a.parent, pmax, pidx, a.out_path, a.out_len, a.out_bonus,
                       reinterpret_cast<unsigned*>(ws));
    return hipGetLastError();
  }
  {
    int W = 0, slice = 0;
    // (tuning/testing: accept_single forces the one-workgroup walk)
    if (!tuning().accept_single && accept_coop_plan(a.batch, a.vocab, device_cu_count(), &W, &slice))
      return launch_accept_coop(a, ws + w.coop, resid, W, slice, stream);
  }
  const double temp = (double)a.temperature;
  hipLaunchKernelGGL(row_reduce_kernel<true>, grid, dim3(256), 0, stream, a.logits, a.vocab, temp, pmax, pidx,
                     psum);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  WalkParams wp;
  wp.walk = dev::alone_params(a, resid);
  wp.nch = nch; wp.pmax = pmax; wp.psum = psum;
  hipLaunchKernelGGL(walk_sample_kernel, dim3(a.batch), dim3(kWalkThreads), 0, stream, wp);
  return hipGetLastError();
}

}  // namespace jk
