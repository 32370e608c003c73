// Internal declarations shared by the library's translation units (not installed).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "jakiro_verify.h"
#include "jk_words.h"

namespace jk {
// The dynamic-LDS limit of a kernel is an attribute it has per device: raised on a device's first launch of
// that kernel (idempotent, so a race between host threads is harmless).  `done` is the caller's static table.
struct LdsLimitRaised {
  bool on_device[64] = {};
};
inline hipError_t raise_lds_limit(const void* kernel, int bytes, LdsLimitRaised& done) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const bool tracked = dev >= 0 && dev < 64;
  if (tracked && done.on_device[dev]) return hipSuccess;
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess && tracked) done.on_device[dev] = true;
  return e;
}
// A launch without the call configuration that <<< >>> pushes and pops (2.45 us of a thread, 2.28 so).  An error is returned, and not left
// for the next hipGetLastError to find.
template <class T>
struct SameType {
  typedef T type;
};
template <class... P>
hipError_t launch_kernel(void (*kernel)(P...), dim3 grid, dim3 threads, unsigned lds, hipStream_t stream, typename SameType<P>::type... args) {
  void* pointers[] = {const_cast<void*>(static_cast<const void*>(&args))...};
  const hipError_t e = hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, threads, pointers, lds, stream);
  if (e != hipSuccess) (void)hipGetLastError();
  return e;
}
}  // namespace jk

namespace jk {

constexpr int kWaveSize = 64;
constexpr int kTileKeys = 32;      // keys per attention tile (one MFMA M-block)
constexpr int kMaxSplits = 64;     // upper bound on KV splits per (sequence, KV head)
constexpr int kMaxTilesPerSplit = 1024;  // so that a split's page ids (paged caches) fit a workgroup's LDS table

// How one attention call is cut into workgroups.  Derived on the host from the
// descriptor and the prefix bound only.
struct AttnPlan {
  int wm;          // 32-row blocks along the query-row axis (8: four waves of two each, tva_wide.hip; else one per wave)
  int wn;          // waves along the key axis (key columns of a round)
  int kt;          // consecutive 32-key tiles a wave takes per round (1 or 2)
  int q_rows;      // query rows per workgroup = 32 * wm
  int n_qtiles;    // workgroups along the query-row axis
  int m_rows;      // T * G query rows per KV head
  int m_pad;       // n_qtiles * q_rows
  int splits;      // KV splits
  int parts;       // partial results per row: the splits, or (fp32) parts of them
  int fused;       // bf16 path: the splits are merged inside the attention kernel (no second launch)
  int ranked;      // bf16 path: sequences taken by falling length, dealt to the XCDs in turn
  int fine;        // bf16 path: partial results in fp32 rather than bf16
  int deep;        // bf16 path, 2x2 waves: the six-tile K/V ring (one workgroup per CU, two rounds in flight)
  size_t part_o_bytes, part_ml_bytes, total_bytes;  // total = header + partials
  size_t covers_bytes;  // what the size query answers: enough for every smaller call as well
};

// Every attention and acceptance workspace starts with a header: 256 bytes whose first word is the
// sticky device error word (jk_last_device_error), then 64-byte lines of synchronisation words for the merges inside the
// attention kernels and the greedy launch (jk_words.h: whose is which).  The header
// must be zero before the first use of a workspace and is kept consistent by the calls themselves.
constexpr size_t kWsErrBytes = 256;
constexpr size_t kAttnHeaderBytes = kWsErrBytes + (size_t)kMaxFusedGroups * 64;  // 32 KiB
static_assert(kAttnHeaderBytes == JK_WORKSPACE_HEADER_BYTES, "public constant");

// Device error bits (public names in jakiro_verify.h)
constexpr unsigned kDevErrBadTree = 1u, kDevErrBadToken = 2u, kDevErrBadPage = 4u, kDevErrMergeWait = 8u,
                   kDevErrWalkWait = 16u;

// Overrides for experiments and tests (jk_set_tuning; seeded once from the JK_* environment
// variables when the library is loaded).  0 / -1 mean "let the library decide".
struct Tuning {
  int attn_wm = 0, attn_wn = 0, attn_splits = 0;
  int attn_fused = -1;     // -1 automatic, 0 never (nor the kernel that cannot do without, tva_wide.hip), 1 whenever the grid allows it; either: a kernel that has one
  int attn_deep = -1;      // six-tile K/V ring of the 2x2 arrangement: -1 automatic, 0 never, 1 whenever one workgroup per CU is planned
  int accept_single = 0;   // 1: one-workgroup sampling walk
  int spin_limit = -1;     // polls of the bounded waits (-1: default)
  // heads and experts by the kernel of equal shares (ring_gemm.hip), linear layers by the one of few columns: -1 automatic, 0 never,
  // 1 wherever they can be
  int ring_gemm = -1, narrow_gemm = -1;
  int verbose = 0;
};
Tuning& tuning();

// whether this device places consecutive workgroups round-robin over its XCDs (checked by jk_init)
bool xcd_placement_verified();

bool make_attn_plan(const jk_attn_desc& d, int max_prefix_len, bool fused_allowed, AttnPlan* plan);

struct AttnArgs {
  const void *q, *k_cache, *v_cache, *k_tree, *v_tree;
  const int32_t* parent;
  const int32_t* prefix_len;
  void* out;
  float* part_o;    // [B*Hkv][splits][m_pad][D], fp32, or bf16 (bf16 path, see AttnPlan::fine)
  float2* part_ml;  // [B*Hkv][splits][m_pad]  (running max in log2 units, sum)
  unsigned* err;    // the workspace's device error word
  unsigned* sync;   // the workspace's group synchronisation words (merge inside the kernel)
  jk_attn_desc d;
  int max_prefix_len;
  float scale_log2;  // softmax scale * log2(e)
  // paged cache (bf16 path only): nullptr / 0 for a contiguous cache
  const int32_t* block_table;
  int max_blocks, page_size, n_pages;
  long long page_stride;
};

hipError_t launch_tva_bf16(const AttnArgs& a, const AttnPlan& p, hipStream_t stream);
hipError_t launch_tva_f32(const AttnArgs& a, const AttnPlan& p, hipStream_t stream);
bool f32_merges(const jk_attn_desc& d, const AttnPlan& pl);  // whether that launch merges the parts of a divided range itself
hipError_t launch_tva_combine(const AttnArgs& a, const AttnPlan& p, hipStream_t stream);

struct AcceptArgs {
  int batch, n_tree, vocab, max_depth, mode;
  float temperature;
  const int32_t *tokens, *parent;
  const float *logits, *draft_probs, *uniforms;
  int32_t *out_path, *out_len, *out_bonus;
  void* workspace;
  // optional indirection: node k of sequence b uses row draft_row[b*n_tree + k] (clamped into
  // [0, n_draft_rows)) of draft_probs instead of row b*n_tree + k
  const int32_t* draft_row;
  long long n_draft_rows;
};
size_t accept_workspace_bytes(int batch, int n_tree, int vocab, int mode);
hipError_t launch_accept(const AcceptArgs& a, hipStream_t stream);
size_t accept_greedy_static_bytes(int batch, int n_tree, int vocab);
hipError_t launch_accept_greedy_static(const AcceptArgs& a, hipStream_t stream);
hipError_t probe_xcd_placement(hipStream_t stream, bool* round_robin);
int device_cu_count();

struct CommitArgs {
  jk_attn_desc d;
  const void *k_tree, *v_tree;
  void *k_cache, *v_cache;
  const int32_t *path, *accept_len;
  int32_t* prefix_len;
  int max_depth, capacity, advance;
  int n_layers;  // 0: the four pointers are the tensors; > 0: device arrays of that many tensor pointers
  // paged caches: nullptr / 0 for contiguous ones
  const int32_t* block_table;
  int max_blocks, page_size, n_pages;
  long long page_stride;
};
hipError_t launch_commit(const CommitArgs& a, hipStream_t stream);

// cooperative sampling walk (several workgroups per tree)
size_t accept_coop_bytes();
bool accept_coop_plan(int batch, int vocab, int cus, int* W, int* slice);
hipError_t launch_accept_coop(const AcceptArgs& a, void* coop_ws, double* resid, int W, int slice, hipStream_t stream);
hipError_t launch_zero_fill(void* p, size_t bytes, hipStream_t stream);
hipError_t launch_stream_read(const void* src, size_t bytes, void* sink, hipStream_t stream);

// few rows times a large weight matrix (stream_gemm.hip): y[m][n] = x[m][k] . w[n][k]^T, fp32, k a multiple of 128
struct StreamGemmArgs {
  const uint16_t *x, *w;  // bf16
  float* y;
  int m, n, k;
  int ksplit;           // parts of the k range; part z writes its partial result y_split elements behind the first one's
  long long y_split;
  // plain products, undivided k range: with `finish` y (or null) and out_bf16 (or null) receive x . w^T + residual (or null)
  bool finish;
  const uint16_t* residual;
  uint16_t* out_bf16;
  // experts: `batch` problems, w_batch elements between their weights; problem e runs for the choices c = 2 r, 2 r + 1 of the
  // rows r of [0, m) with sel[c] == e, or not at all.  Rows of y, of act and of the down projection's x are numbered by
  // choice, so that no kernel has to find out how many rows before r chose the same expert; x of gate and up has the rows r
  int batch;
  long long w_batch;
  const int* sel;
  const uint16_t* w2;   // gate and up projections in one launch: w, y and w2, y2; or, with `act` (undivided k range),
  float* y2;            // act[choice][n] = silu(x . w^T) * (x . w2^T) in bf16
  uint16_t* act;
  // output heads: row 2 r + h of the product's left side is made of rows 2 r and 2 r + 1 of x, token r's two features f1 and
  // f2 with router scores s1 and s2 = s_top[2 r], s_top[2 r + 1]: s_(h + 1) f_(h + 1) (JK_HEADS_DECOUPLED), or
  // s1 f1 + s2 f2 (h = 0) and beta f1 - alpha f2 (h = 1)
  const float* s_top;
  int heads_mode;
  float alpha, beta;
  // output heads, undivided k range: or null, [m][blocks of kStatColumns columns]: a block's maximum and sum of exp((x - maximum) inv_temp)
  float2* stats;
  float scale_hi, scale_lo;  // inv_temp log2(e), in two parts
};
constexpr int kStatColumns = 128;
int stream_gemm_ksplit(int m, int n, int k, int batch, bool pair, int split_ns, double* ns = nullptr);
hipError_t launch_stream_gemm(const StreamGemmArgs& p, hipStream_t stream);       // m <= 256
// plain products with `finish` of few rows and columns, in one launch
struct NarrowPlan {
  int strip, strips, rows, blocks, parts;  // weight rows of a workgroup, strips, rows of X, blocks of those, parts of k (1 or 2; 0: not possible)
  double ns;
};
NarrowPlan narrow_plan(int m, int n, int k);
size_t narrow_gemm_bytes(const NarrowPlan& plan);
hipError_t launch_narrow_gemm(const StreamGemmArgs& p, const NarrowPlan& plan, void* workspace, hipStream_t stream);
unsigned long long meeting_tag();  // another one for every launch (see dev::second_to_meet)
hipError_t launch_stream_gemm_heads(const StreamGemmArgs& p, hipStream_t stream);  // m <= 64
hipError_t launch_stream_gemm_pair(const StreamGemmArgs& p, hipStream_t stream);  // m <= 128
hipError_t launch_stream_gemm_down(const StreamGemmArgs& p, hipStream_t stream);  // m <= 128
// the same products with equal shares of the weight rows.  rows: how many an expert is likely to have at most (others take
// several passes over its weights), items: how many experts are likely to be chosen
constexpr int kRingRows = 32;  // of X at a time
struct RingExperts {
  double mean;       // rows of an expert
  bool many;         // more than kRingRows of them, mostly
  int likely, most;  // experts that are chosen
};
bool ring_gemm_takes_heads(int m, int n);
bool ring_gemm_takes_pair(const RingExperts& x, int d_ff, int d_model);
bool ring_gemm_takes_down(const RingExperts& x, int d_model, int d_ff);
hipError_t launch_ring_gemm_heads(const StreamGemmArgs& p, hipStream_t stream);
hipError_t launch_ring_gemm_pair(const StreamGemmArgs& p, int rows, int items, hipStream_t stream);
hipError_t launch_ring_gemm_down(const StreamGemmArgs& p, int rows, int items, hipStream_t stream);

// draft head step (two heads over the shared output embedding)
struct DraftHeadsArgs {
  int rows, d_model, vocab, top_k, mode;
  float temperature, alpha, beta;
  const void *f_top, *w_head;
  const float* s_top;
  float *logits, *draft_probs, *topk_probs;
  int32_t* topk_tokens;
  void* workspace;
  size_t workspace_bytes;
};
size_t draft_heads_workspace_bytes(int rows, int d_model, int vocab);
size_t draft_heads_least_bytes(int rows, int d_model, int vocab);  // without which a call is refused
hipError_t launch_draft_heads(const DraftHeadsArgs& a, hipStream_t stream);

// router + expert MLPs of the draft layer
struct MoeArgs {
  int rows, d_model, d_ff, n_experts;
  const void *u, *centroids, *w_gate, *w_up, *w_down;
  void *f_top, *f_mix;
  float* s_top;
  int32_t* expert_idx;
  void* workspace;
};
size_t moe_experts_workspace_bytes(int rows, int d_model, int d_ff, int n_experts);
hipError_t launch_moe_experts(const MoeArgs& a, hipStream_t stream);

// draft tree growth
struct TreeGrowArgs {
  int batch, n_front, top_k, width, max_nodes, q_row_base;
  int32_t *tokens, *parent, *q_row, *n_nodes;  // state [batch][max_nodes], [batch]
  float* score;
  const int32_t* frontier_in;  // [batch][n_front] or null (the root)
  const int32_t* cand_tok;     // [batch*n_front][2][top_k]
  const float* cand_p;
  int32_t* frontier_out;       // [batch][width]
  unsigned mg_top_k = 0;       // 2^16 / top_k + 1: c / top_k == (c * mg_top_k) >> 16 for c and top_k up to 256
};
struct TreeFinalArgs {
  int batch, n_keep, max_nodes;
  const int32_t *tokens, *parent, *q_row, *n_nodes;
  const float* score;
  int32_t *out_tokens, *out_parent, *out_q_row, *out_old, *n_valid;
};
int tree_max_nodes();
hipError_t launch_tree_grow(const TreeGrowArgs& a, hipStream_t stream);
hipError_t launch_tree_grow_tail(const TreeGrowArgs& a, int k1, int k2, hipStream_t stream);
hipError_t launch_tree_fill_static(const TreeGrowArgs& a, const int* slot, const int* expert, const int* rank, int n_new,
                                   const int* next_index, int n_next, int* new_ids, hipStream_t stream);
hipError_t launch_tree_reset(int32_t* n_nodes, int batch, hipStream_t stream);  // no nodes in any sequence
hipError_t launch_tree_finalize(const TreeFinalArgs& a, hipStream_t stream);
hipError_t launch_gather_rows(const float* q_all, const int* q_row, float* out, long long n_nodes, int vocab,
                              long long n_q_rows, hipStream_t stream);

// plain linear layer
struct LinearArgs {
  int m, n, k;
  const void *x, *w, *residual;
  float* out_f32;
  void* out_bf16;
  void* workspace;
};
size_t linear_workspace_bytes(int m, int n, int k);

// what one call of these sizes needs, 0 where it is not supported (the public size queries cover fewer rows as well)
size_t draft_heads_call_bytes(int rows, int d_model, int vocab);
size_t moe_experts_call_bytes(const jk_moe_desc& d);
size_t linear_call_bytes(int m, int n, int k);
bool linear_call_writes(int m, int n, int k);  // whether such a call uses its workspace
// jk_linear with a workspace of linear_call_bytes, or none where the call uses none
jk_status linear_call(int m, int n, int k, const void* x, const void* w, const void* residual, void* out_bf16, float* out_f32,
                      void* workspace, void* hip_stream);
hipError_t launch_linear(const LinearArgs& a, hipStream_t stream);

}  // namespace jk
