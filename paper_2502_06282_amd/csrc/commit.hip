// Commit of the accepted path to the KV cache of one layer (gfx950).
//
// What it computes (Section 2.1 step 3 of the paper: accepted tokens are
// appended to the sequence, the rest of the draft is dropped): the key/value
// rows of the accepted tree nodes, in path order, become the next rows of the
// cache.  A plain gather-copy: one workgroup per (layer, sequence, path
// position) moves that node's K and V rows of all KV heads with 16-byte
// accesses; the layers of a model go in one launch (the copy is a few tens of
// KB per layer, so a launch per layer would cost more than the copies).  The
// prefix length is advanced by a second, tiny kernel, because every workgroup
// of the first still reads the old value.
//
// What bounds it: two launches and the trips to memory in each, of which the first kernel makes two (path, lengths and the
// layer's pointers together; the rows) and the second one: a wave looks at 64 entries of a path at once.  With the entries
// looked at one by one, three trips more, and flat accesses through the layers' pointers ten drawn verification steps took 1.009 times as
// long (42.5 us for four layers, 41.7 like this).  Rows stored through to memory: no faster.
#include "jk_internal.h"

namespace jk {
namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

struct CommitParams {
  const unsigned char *kt, *vt;    // one layer: the tensors; several layers: device arrays of n_layers pointers
  unsigned char *kc, *vc;
  const int32_t *path, *accept_len;
  int32_t* prefix_len;
  int T, Hkv, max_depth, capacity;
  int row_chunks;                  // 16-byte chunks per (node, KV head) row
  long long kc_sb, kc_sl, kc_sh, kt_sb, kt_st, kt_sh;  // strides in bytes
  // paged caches: kc / vc are page pools and position t of sequence b lives in page
  // block_table[b * max_blocks + t / page_size], slot t % page_size
  const int32_t* block_table;
  int max_blocks, page_size, n_pages;
  long long page_sb;  // page stride in bytes
  unsigned long long mg_depth, mg_chunks;  // for x / max_depth and c / row_chunks (see quotient), or 0
};
typedef __attribute__((address_space(1))) unsigned char device_byte;
typedef __attribute__((address_space(1))) u32x4 device_u32x4;

// n / d by floor(2^32 / d) + 1, which is exact while n * d < 2^32, or, without it, by division
__device__ __forceinline__ int quotient(unsigned n, unsigned d, unsigned long long mg) { return mg ? (int)((n * mg) >> 32) : (int)(n / d); }
unsigned long long magic(long long largest, int d) { return largest * d < (1LL << 32) ? (1ull << 32) / (unsigned)d + 1ull : 0ull; }

// rows of sequence b that are committed: accept_len cut to [0, max_depth], ended in front of
// the first node id outside [0, T), and limited to the room left in the cache.  By a wave, all its lanes; `node`: the path's
// entry at `lane`, asked for by the caller beside the lengths
__device__ __forceinline__ int path_entry(const CommitParams& p, int b, int i) { return p.path[(long long)b * p.max_depth + min(i, p.max_depth - 1)]; }
__device__ __forceinline__ int committed_rows(const CommitParams& p, int b, int L, int accepted, int node, int lane) {
  const int most = accepted < 0 ? 0 : (accepted > p.max_depth ? p.max_depth : accepted);
  int n = most;
  for (int at = 0; at < most; at += 64) {
    if (at) node = path_entry(p, b, at + lane);
    const unsigned long long bad = __ballot(node < 0 || node >= p.T);
    if (bad) {
      n = min(at + __ffsll((long long)bad) - 1, most);
      break;
    }
  }
  const int room = p.capacity - L;
  return n < room ? n : (room > 0 ? room : 0);
}

// grid: x = sequence * max_depth + path position, y = layer
template <bool LAYERS>
__global__ __launch_bounds__(256) void commit_rows_kernel(CommitParams p) {
  const int b = quotient(blockIdx.x, p.max_depth, p.mg_depth), i = (int)blockIdx.x - b * p.max_depth, lane = threadIdx.x & 63;
  // All of it asked for before any of it is waited for, by vector loads: scalar ones are waited for in batches, and left alone
  // the compiler asks where it uses.
  int zero = 0;
  asm volatile("" : "+v"(zero));
  int entry = path_entry(p, b, lane), node = path_entry(p, b, i + zero), length = p.prefix_len[b + zero], accepted = p.accept_len[b + zero];
  unsigned long long kt = (unsigned long long)p.kt, vt = (unsigned long long)p.vt, kc = (unsigned long long)p.kc, vc = (unsigned long long)p.vc;
  if (LAYERS) {
    const int y = (int)blockIdx.y + zero;
    kt = reinterpret_cast<const unsigned long long*>(p.kt)[y];
    vt = reinterpret_cast<const unsigned long long*>(p.vt)[y];
    kc = reinterpret_cast<const unsigned long long*>(p.kc)[y];
    vc = reinterpret_cast<const unsigned long long*>(p.vc)[y];
    asm volatile("" : "+v"(entry), "+v"(node), "+v"(length), "+v"(accepted), "+v"(kt), "+v"(vt), "+v"(kc), "+v"(vc));
  } else {
    asm volatile("" : "+v"(entry), "+v"(node), "+v"(length), "+v"(accepted));
  }
  auto uniform = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
  node = uniform(node);
  accepted = uniform(accepted);
  const int L = max(uniform(length), 0);
  if (i >= committed_rows(p, b, L, accepted, entry, lane)) return;
  const long long src = b * p.kt_sb + node * p.kt_st;
  long long dst = b * p.kc_sb + (long long)(L + i) * p.kc_sl;
  if (p.block_table) {
    const int pos = L + i, pi = pos / p.page_size;  // pi < max_blocks: pos < capacity <= max_blocks * page_size
    int page = p.block_table[(long long)b * p.max_blocks + pi];
    page = page < 0 ? 0 : (page >= p.n_pages ? p.n_pages - 1 : page);
    dst = page * p.page_sb + (long long)(pos - pi * p.page_size) * p.kc_sl;
  }
  device_byte *ks = (device_byte*)(kt + src), *vs = (device_byte*)(vt + src), *kd = (device_byte*)(kc + dst), *vd = (device_byte*)(vc + dst);
  const int total = p.Hkv * p.row_chunks;
  for (int c = threadIdx.x; c < total; c += 256) {
    const int h = quotient(c, p.row_chunks, p.mg_chunks), o = (c - h * p.row_chunks) * 16;
    const u32x4 kv = *reinterpret_cast<const device_u32x4*>(ks + h * p.kt_sh + o);
    const u32x4 vv = *reinterpret_cast<const device_u32x4*>(vs + h * p.kt_sh + o);
    *reinterpret_cast<device_u32x4*>(kd + h * p.kc_sh + o) = kv;
    *reinterpret_cast<device_u32x4*>(vd + h * p.kc_sh + o) = vv;
  }
}

// A wave per sequence
__global__ __launch_bounds__(64) void advance_len_kernel(CommitParams p) {
  const int b = blockIdx.x, lane = threadIdx.x;
  int zero = 0;
  asm volatile("" : "+v"(zero));  // (as above)
  int entry = path_entry(p, b, lane), length = p.prefix_len[b + zero], accepted = p.accept_len[b + zero];
  asm volatile("" : "+v"(entry), "+v"(length), "+v"(accepted));
  accepted = __builtin_amdgcn_readfirstlane(accepted);
  const int L = max(__builtin_amdgcn_readfirstlane(length), 0);
  const int n = committed_rows(p, b, L, accepted, entry, lane);
  if (lane == 0) p.prefix_len[b] = L + n;
}

}  // namespace

hipError_t launch_commit(const CommitArgs& a, hipStream_t stream) {
  const jk_attn_desc& d = a.d;
  const long long es = d.dtype == JK_BF16 ? 2 : 4;
  CommitParams p;
  p.kt = static_cast<const unsigned char*>(a.k_tree);
  p.vt = static_cast<const unsigned char*>(a.v_tree);
  p.kc = static_cast<unsigned char*>(a.k_cache);
  p.vc = static_cast<unsigned char*>(a.v_cache);
  p.path = a.path; p.accept_len = a.accept_len; p.prefix_len = a.prefix_len;
  p.T = d.n_tree; p.Hkv = d.n_kv_heads; p.max_depth = a.max_depth; p.capacity = a.capacity;
  p.row_chunks = (int)(d.head_dim * es / 16);
  p.kc_sb = d.kc_stride_b * es; p.kc_sl = d.kc_stride_l * es; p.kc_sh = d.kc_stride_h * es;
  p.kt_sb = d.kt_stride_b * es; p.kt_st = d.kt_stride_t * es; p.kt_sh = d.kt_stride_h * es;
  p.block_table = a.block_table; p.max_blocks = a.max_blocks; p.page_size = a.page_size; p.n_pages = a.n_pages;
  p.page_sb = a.page_stride * es;
  p.mg_depth = magic((long long)d.batch * a.max_depth, a.max_depth);
  p.mg_chunks = magic((long long)d.n_kv_heads * p.row_chunks, p.row_chunks);
  const dim3 grid((unsigned)(d.batch * a.max_depth), (unsigned)(a.n_layers > 0 ? a.n_layers : 1));
  if (a.n_layers > 0)
    hipLaunchKernelGGL(commit_rows_kernel<true>, grid, dim3(256), 0, stream, p);
  else
    hipLaunchKernelGGL(commit_rows_kernel<false>, grid, dim3(256), 0, stream, p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !a.advance) return e;
  hipLaunchKernelGGL(advance_len_kernel, dim3((unsigned)d.batch), dim3(64), 0, stream, p);
  return hipGetLastError();
}

}  // namespace jk
