"""Python binding of libjakiro_verify (argument marshalling only).

Function names and argument meaning follow include/jakiro_verify.h.  Tensors
are torch tensors on the ROCm device; torch is used for device memory and the
current stream, nothing else.  The calls that a decoding loop makes are marshalled
by the extension module `_native` (csrc/native.cpp): this file gives them their
names, defaults and documentation.  Size queries, plans and the other host-only
entry points go through ctypes.
"""
from __future__ import annotations

import ctypes
import os
from typing import Optional, Tuple

_HERE = os.path.dirname(os.path.abspath(__file__))
_LIB_PATH = os.path.join(_HERE, "libjakiro_verify.so")

JK_BF16, JK_F32 = 0, 1
JK_GREEDY, JK_SAMPLE = 0, 1
JK_DEVERR_BAD_TREE, JK_DEVERR_BAD_TOKEN, JK_DEVERR_BAD_PAGE, JK_DEVERR_MERGE_WAIT, JK_DEVERR_WALK_WAIT = 1, 2, 4, 8, 16
JK_WORKSPACE_HEADER_BYTES = 32768
JK_HEADS_DECOUPLED, JK_HEADS_CONTRASTIVE = 0, 1
MAX_TREE = 128


class JakiroError(RuntimeError):
    def __init__(self, status: int, where: str):
        self.status = status
        super().__init__(f"{where}: {lib().jk_status_string(status).decode()} (status {status})")


class AttnDesc(ctypes.Structure):
    _fields_ = [
        ("batch", ctypes.c_int32), ("n_tree", ctypes.c_int32), ("n_q_heads", ctypes.c_int32),
        ("n_kv_heads", ctypes.c_int32), ("head_dim", ctypes.c_int32),
        ("q_stride_b", ctypes.c_int64), ("q_stride_t", ctypes.c_int64), ("q_stride_h", ctypes.c_int64),
        ("kc_stride_b", ctypes.c_int64), ("kc_stride_l", ctypes.c_int64), ("kc_stride_h", ctypes.c_int64),
        ("kt_stride_b", ctypes.c_int64), ("kt_stride_t", ctypes.c_int64), ("kt_stride_h", ctypes.c_int64),
        ("o_stride_b", ctypes.c_int64), ("o_stride_t", ctypes.c_int64), ("o_stride_h", ctypes.c_int64),
        ("scale", ctypes.c_float), ("dtype", ctypes.c_int32),
    ]


_lib = None

class DraftHeadsDesc(ctypes.Structure):
    """jk_draft_heads_desc"""
    _fields_ = [("rows", ctypes.c_int32), ("d_model", ctypes.c_int32), ("vocab", ctypes.c_int32),
                ("top_k", ctypes.c_int32), ("mode", ctypes.c_int32), ("temperature", ctypes.c_float),
                ("alpha", ctypes.c_float), ("beta", ctypes.c_float)]


class MoeDesc(ctypes.Structure):
    """jk_moe_desc"""
    _fields_ = [("rows", ctypes.c_int32), ("d_model", ctypes.c_int32), ("d_ff", ctypes.c_int32),
                ("n_experts", ctypes.c_int32)]


class TreeStateDesc(ctypes.Structure):
    """jk_tree_state"""
    _fields_ = [("tokens", ctypes.c_void_p), ("parent", ctypes.c_void_p), ("score", ctypes.c_void_p),
                ("q_row", ctypes.c_void_p), ("n_nodes", ctypes.c_void_p), ("max_nodes", ctypes.c_int32)]


class PagedKV(ctypes.Structure):
    """jk_paged_kv"""
    _fields_ = [("block_table", ctypes.c_void_p), ("max_blocks", ctypes.c_int32), ("page_size", ctypes.c_int32),
                ("n_pages", ctypes.c_int32), ("page_stride", ctypes.c_int64)]


EXPORTS = ("jk_tree_verify_attention_workspace", "jk_tree_verify_attention_plan", "jk_tree_verify_attention", "jk_tree_verify_attention_paged",
           "jk_commit_path_layers_paged", "jk_accept_path_workspace",
           "jk_accept_path", "jk_accept_path_greedy_static", "jk_accept_path_rows", "jk_draft_heads_workspace", "jk_draft_heads", "jk_moe_experts_workspace", "jk_moe_experts", "jk_linear_workspace", "jk_linear", "jk_tree_grow", "jk_tree_grow_tail", "jk_tree_fill_static", "jk_tree_finalize", "jk_gather_draft_probs", "jk_commit_path", "jk_commit_path_layers", "jk_workspace_init", "jk_init", "jk_set_tuning", "jk_last_device_error", "jk_stream_read_probe", "jk_validate_tree", "jk_status_string", "jk_version")


def library_path() -> str:
    return _LIB_PATH


def lib() -> ctypes.CDLL:
    """The loaded library; raises if it has not been built (no fallback path exists)."""
    global _lib
    if _lib is None:
        if not os.path.exists(_LIB_PATH):
            raise RuntimeError(f"{_LIB_PATH} is missing: build it with "
                               "`python -m paper_2502_06282_amd.build` (needs hipcc)")
        l = ctypes.CDLL(_LIB_PATH)
        vp, i32, sz = ctypes.c_void_p, ctypes.c_int32, ctypes.c_size_t
        l.jk_tree_verify_attention_workspace.restype = sz
        l.jk_tree_verify_attention_workspace.argtypes = [ctypes.POINTER(AttnDesc), i32]
        l.jk_tree_verify_attention.restype = i32
        l.jk_tree_verify_attention.argtypes = [ctypes.POINTER(AttnDesc), vp, vp, vp, vp, vp, vp, vp, i32,
                                               vp, vp, sz, vp]
        l.jk_tree_verify_attention_paged.restype = i32
        l.jk_tree_verify_attention_paged.argtypes = [ctypes.POINTER(AttnDesc), ctypes.POINTER(PagedKV), vp, vp, vp, vp, vp,
                                                     vp, vp, i32, vp, vp, sz, vp]
        l.jk_commit_path_layers_paged.restype = i32
        l.jk_commit_path_layers_paged.argtypes = [ctypes.POINTER(AttnDesc), ctypes.POINTER(PagedKV), i32, vp, vp, vp, vp,
                                                  vp, vp, i32, vp, i32, vp]
        l.jk_accept_path_workspace.restype = sz
        l.jk_accept_path_workspace.argtypes = [i32, i32, i32, i32]
        l.jk_accept_path.restype = i32
        l.jk_accept_path.argtypes = [i32, i32, i32, i32, vp, vp, vp, i32, ctypes.c_float, vp, vp, vp, vp,
                                     vp, vp, sz, vp]
        l.jk_accept_path_rows.restype = i32
        l.jk_accept_path_rows.argtypes = [i32, i32, i32, i32, vp, vp, vp, i32, ctypes.c_float, vp, ctypes.c_int64, vp,
                                          vp, vp, vp, vp, vp, sz, vp]
        l.jk_commit_path.restype = i32
        l.jk_commit_path.argtypes = [ctypes.POINTER(AttnDesc), vp, vp, vp, vp, vp, vp, i32, i32, vp, i32, vp]
        l.jk_commit_path_layers.restype = i32
        l.jk_commit_path_layers.argtypes = [ctypes.POINTER(AttnDesc), i32, vp, vp, vp, vp, vp, vp, i32, i32, vp, i32, vp]
        l.jk_draft_heads_workspace.restype = sz
        l.jk_draft_heads_workspace.argtypes = [i32, i32, i32]
        l.jk_draft_heads.restype = i32
        l.jk_draft_heads.argtypes = [ctypes.POINTER(DraftHeadsDesc), vp, vp, vp, vp, vp, vp, vp, vp, sz, vp]
        l.jk_moe_experts_workspace.restype = sz
        l.jk_moe_experts_workspace.argtypes = [ctypes.POINTER(MoeDesc)]
        l.jk_moe_experts.restype = i32
        l.jk_moe_experts.argtypes = [ctypes.POINTER(MoeDesc), vp, vp, vp, vp, vp, vp, vp, vp, vp, vp, sz, vp]
        l.jk_linear_workspace.restype = sz
        l.jk_linear_workspace.argtypes = [i32, i32, i32]
        l.jk_linear.restype = i32
        l.jk_linear.argtypes = [i32, i32, i32, vp, vp, vp, vp, vp, vp, sz, vp]
        l.jk_tree_grow.restype = i32
        l.jk_tree_grow.argtypes = [ctypes.POINTER(TreeStateDesc), i32, i32, i32, i32, i32, vp, vp, vp, vp, vp]
        l.jk_tree_grow_tail.restype = i32
        l.jk_tree_grow_tail.argtypes = [ctypes.POINTER(TreeStateDesc), i32, i32, i32, i32, i32, i32, i32, vp, vp, vp, vp]
        l.jk_tree_fill_static.restype = i32
        l.jk_tree_fill_static.argtypes = [ctypes.POINTER(TreeStateDesc), i32, i32, i32, i32, vp, vp, vp, vp, vp, vp, i32,
                                          vp, i32, vp, vp, vp]
        l.jk_tree_finalize.restype = i32
        l.jk_tree_finalize.argtypes = [ctypes.POINTER(TreeStateDesc), i32, i32, vp, vp, vp, vp, vp, vp]
        l.jk_gather_draft_probs.restype = i32
        l.jk_gather_draft_probs.argtypes = [i32, i32, i32, vp, ctypes.c_int64, vp, vp, vp]
        l.jk_workspace_init.restype = i32
        l.jk_workspace_init.argtypes = [vp, sz, vp]
        l.jk_tree_verify_attention_plan.restype = i32
        l.jk_tree_verify_attention_plan.argtypes = [ctypes.POINTER(AttnDesc), i32, ctypes.POINTER(i32)]
        l.jk_init.restype = i32
        l.jk_init.argtypes = [vp]
        l.jk_set_tuning.restype = i32
        l.jk_set_tuning.argtypes = [ctypes.c_char_p, i32]
        l.jk_last_device_error.restype = i32
        l.jk_last_device_error.argtypes = [vp]
        l.jk_stream_read_probe.restype = i32
        l.jk_stream_read_probe.argtypes = [vp, sz, vp, vp]
        l.jk_validate_tree.restype = i32
        l.jk_validate_tree.argtypes = [ctypes.POINTER(ctypes.c_int32), i32]
        l.jk_status_string.restype = ctypes.c_char_p
        l.jk_status_string.argtypes = [i32]
        l.jk_version.restype = ctypes.c_char_p
        l.jk_version.argtypes = []
        _lib = l
    return _lib


class _NotBuilt:
    """Stands in for `_native` until the extension has been built (no fallback path exists)."""

    def __getattr__(self, name):
        global _n
        import importlib
        import torch  # noqa: F401  (the extension links against torch's libraries)
        try:
            _n = importlib.import_module("._native", __package__)
        except ImportError as e:
            raise RuntimeError(f"{os.path.join(_HERE, '_native.so')} cannot be loaded ({e}): build it with "
                               "`python -m paper_2502_06282_amd.build` (needs hipcc)") from e
        _n.set_error_class(JakiroError)
        return getattr(_n, name)


_n = _NotBuilt()


def __getattr__(name):
    if name == "PreparedCall":  # a call with its arguments marshalled once (returned by the prepare_* functions)
        return _n.PreparedCall
    raise AttributeError(name)


def version() -> str:
    return lib().jk_version().decode()


def validate_tree(parent) -> int:
    """Status code of jk_validate_tree for a host sequence of ints."""
    arr = (ctypes.c_int32 * len(parent))(*[int(x) for x in parent])
    return int(lib().jk_validate_tree(arr, len(parent)))


def _ptr(t) -> Optional[int]:
    return None if t is None else t.data_ptr()


def _stream_handle(stream) -> Optional[int]:
    """The hipStream_t of `stream` (default: torch's current stream).  The first use on a device also runs
    jk_init there (a short synchronous probe), unless that stream is being captured into a graph."""
    return _n.stream_handle(stream) or None


def _new_workspace(nbytes: int, device, stream):
    """A zero-filled workspace whose fill is ordered on the stream the library call will use, and which the
    caching allocator will not hand out again while that stream may still be using it."""
    import torch
    s = torch.cuda.current_stream(device) if stream is None else stream
    with torch.cuda.stream(s):
        ws = torch.zeros(nbytes, dtype=torch.uint8, device=device)
    ws.record_stream(s)
    return ws


def set_tuning(name: str, value: int) -> None:
    """jk_set_tuning: force part of a launch plan (experiments and tests)."""
    st = lib().jk_set_tuning(name.encode(), int(value))
    if st != 0:
        raise JakiroError(st, f"jk_set_tuning({name})")


def last_device_error(workspace) -> int:
    """jk_last_device_error: the sticky JK_DEVERR_* bits of an attention or acceptance workspace (synchronous)."""
    return int(lib().jk_last_device_error(_ptr(workspace)))


def _make_desc(q, k_cache, k_tree, out, scale: float) -> AttnDesc:
    import torch
    B, T, Hq, D = q.shape
    Hkv = k_tree.shape[2]
    if q.dtype == torch.bfloat16:
        dt = JK_BF16
    elif q.dtype == torch.float32:
        dt = JK_F32
    else:
        raise TypeError("q must be bfloat16 or float32")
    for t in (q, k_cache, k_tree, out):
        if t is not None and t.stride(-1) != 1 and t.shape[-1] > 1:
            raise ValueError("head_dim must be the contiguous innermost axis")
    kc = k_cache.stride() if k_cache is not None else (0, 0, 0, 1)
    return AttnDesc(B, T, Hq, Hkv, D, q.stride(0), q.stride(1), q.stride(2), kc[0], kc[1], kc[2],
                    k_tree.stride(0), k_tree.stride(1), k_tree.stride(2),
                    out.stride(0), out.stride(1), out.stride(2), float(scale), dt)


def tree_verify_attention_workspace(q, k_cache, k_tree, max_prefix_len: int, scale: float = 0.0) -> int:
    d = _make_desc(q, k_cache, k_tree, q, scale)
    return int(lib().jk_tree_verify_attention_workspace(ctypes.byref(d), int(max_prefix_len)))


def tree_verify_attention_plan(q, k_cache, k_tree, max_prefix_len: int, scale: float = 0.0) -> dict:
    """jk_tree_verify_attention_plan as a dict (wm, wn, kt, row_tiles, splits, fused)."""
    _stream_handle(None)  # (the plan depends on jk_init having run on this device)
    d = _make_desc(q, k_cache, k_tree, q, scale)
    out = (ctypes.c_int32 * 6)()
    st = lib().jk_tree_verify_attention_plan(ctypes.byref(d), int(max_prefix_len), out)
    if st != 0:
        raise JakiroError(st, "jk_tree_verify_attention_plan")
    return dict(zip(("wm", "wn", "kt", "row_tiles", "splits", "fused"), [int(v) for v in out]))


def tree_verify_attention(q, k_cache, v_cache, k_tree, v_tree, parent, prefix_len,
                          max_prefix_len: Optional[int] = None, scale: float = 0.0, out=None,
                          workspace=None, stream=None):
    """jk_tree_verify_attention.  q [B,T,Hq,D]; k_cache, v_cache [B,Lcap,Hkv,D] (same strides);
    k_tree, v_tree [B,T,Hkv,D] (same strides); parent int32 [B,T]; prefix_len int32 [B], all on
    the device.  Returns out [B,T,Hq,D] (allocated unless given).  Asynchronous on `stream`
    (default: torch's current stream)."""
    if workspace is None:
        kc = None if k_cache is None or k_cache.shape[1] == 0 else k_cache
        bound = max_prefix_len if max_prefix_len is not None else 0 if kc is None else int(kc.shape[1])
        need = int(lib().jk_tree_verify_attention_workspace(ctypes.byref(_make_desc(q, kc, k_tree, q if out is None else out, scale)),
                                                            int(bound)))
        if need == 0:
            raise JakiroError(3, "jk_tree_verify_attention_workspace")
        workspace = _new_workspace(need, q.device, stream)
    return _n.attention(q, k_cache, v_cache, None, k_tree, v_tree, parent, prefix_len, max_prefix_len, scale, out, workspace, stream)


def accept_path_workspace(batch: int, n_tree: int, vocab: int, mode: int) -> int:
    return int(lib().jk_accept_path_workspace(batch, n_tree, vocab, mode))


def stream_read_probe(src, sink, stream=None) -> None:
    """jk_stream_read_probe over the whole tensor `src` (measurement aid)."""
    st = lib().jk_stream_read_probe(_ptr(src), src.numel() * src.element_size(), _ptr(sink), _stream_handle(stream))
    if st != 0:
        raise JakiroError(st, "jk_stream_read_probe")


def workspace_init(workspace, stream=None) -> None:
    """jk_workspace_init: zero-fill a workspace tensor on `stream` (once, before its first accept_path)."""
    st = lib().jk_workspace_init(_ptr(workspace), workspace.numel() * workspace.element_size(),
                                 _stream_handle(stream))
    if st != 0:
        raise JakiroError(st, "jk_workspace_init")


def accept_path(tree_tokens, parent, target_logits, mode: int = JK_GREEDY, temperature: float = 1.0,
                draft_probs=None, uniforms=None, max_depth: Optional[int] = None, workspace=None,
                stream=None) -> Tuple["torch.Tensor", "torch.Tensor", "torch.Tensor"]:
    """jk_accept_path.  tree_tokens, parent int32 [B,N]; target_logits fp32 [B,N+1,V] contiguous;
    sampling also needs draft_probs fp32 [B,N,V] and uniforms fp32 [B,N+1].
    Returns (path [B,max_depth], accept_len [B], bonus_token [B]) int32 device tensors."""
    if workspace is None:
        B, N = tree_tokens.shape
        need = accept_path_workspace(B, N, target_logits.shape[-1], mode)
        if need == 0:
            raise JakiroError(3, "jk_accept_path_workspace")
        workspace = _new_workspace(need, tree_tokens.device, stream)
    return _n.accept(tree_tokens, parent, target_logits, mode, temperature, draft_probs, None, uniforms, max_depth, workspace, stream)


def accept_path_greedy_static(tree_tokens, parent, target_logits, out_path, out_accept_len, out_bonus_token,
                              stream=None) -> None:
    """jk_accept_path_greedy_static: greedy acceptance without a workspace (the library's built-in scratch
    buffer); the caller passes every output tensor, the call allocates nothing.  out_path int32 [B, max_depth]."""
    import torch
    B, N = tree_tokens.shape
    V = target_logits.shape[-1]
    for t in (tree_tokens, parent, out_path, out_accept_len, out_bonus_token):
        if t.dtype != torch.int32 or not t.is_contiguous():
            raise TypeError("tokens, parent and the outputs must be contiguous int32")
    if target_logits.dtype != torch.float32 or not target_logits.is_contiguous() or target_logits.shape != (B, N + 1, V):
        raise TypeError("target_logits must be contiguous float32 [B, N+1, V]")
    if out_path.dim() != 2 or out_path.shape[0] != B or out_accept_len.numel() != B or out_bonus_token.numel() != B:
        raise ValueError("outputs must be [B, max_depth], [B], [B]")
    fn = lib().jk_accept_path_greedy_static
    vp, i32 = ctypes.c_void_p, ctypes.c_int32
    fn.restype = i32
    fn.argtypes = [i32, i32, i32, i32, vp, vp, vp, vp, vp, vp, vp]
    st = fn(B, N, V, int(out_path.shape[1]), _ptr(tree_tokens), _ptr(parent), _ptr(target_logits), _ptr(out_path),
            _ptr(out_accept_len), _ptr(out_bonus_token), _stream_handle(stream))
    if st != 0:
        raise JakiroError(st, "jk_accept_path_greedy_static")


def prepare_tree_verify_attention(q, k_cache, v_cache, k_tree, v_tree, parent, prefix_len, out, workspace,
                                  max_prefix_len: Optional[int] = None, scale: float = 0.0) -> "PreparedCall":
    """Same arguments as tree_verify_attention with out and workspace given; nothing is launched.  Returns a call whose
    `launch(stream=None)` issues exactly that one library call: what a decoding loop, or a HIP-graph capture of it, calls
    per step.  It holds references to every tensor it points to."""
    return _n.prepare_attention(q, k_cache, v_cache, None, k_tree, v_tree, parent, prefix_len, max_prefix_len, scale, out, workspace)


def commit_path(k_tree, v_tree, k_cache, v_cache, path, accept_len, prefix_len, advance: bool = True,
                stream=None) -> None:
    """jk_commit_path: copies the K/V rows of the accepted nodes path[b][:accept_len[b]] to the cache
    positions prefix_len[b]..., in place; advances prefix_len (device int32 [B]) when `advance`."""
    _n.commit(k_tree, v_tree, k_cache, v_cache, None, path, accept_len, prefix_len, advance, 0, stream)


def prepare_commit_path(k_tree, v_tree, k_cache, v_cache, path, accept_len, prefix_len,
                        advance: bool = True) -> "PreparedCall":
    """Same arguments as commit_path; nothing is launched."""
    return _n.prepare_commit(k_tree, v_tree, k_cache, v_cache, None, path, accept_len, prefix_len, advance, 0)


def prepare_commit_path_layers(k_trees, v_trees, k_caches, v_caches, path, accept_len, prefix_len,
                               advance: bool = True) -> "PreparedCall":
    """jk_commit_path_layers for lists of per-layer tensors (all of one shape, dtype and stride set): builds the
    device pointer tables once; `launch()` commits every layer with one call."""
    import torch
    n = len(k_trees)
    for ts in (k_trees, v_trees, k_caches, v_caches):
        if len(ts) != n or any(t.stride() != ts[0].stride() or t.shape != ts[0].shape for t in ts):
            raise ValueError("per-layer tensors must share shape and strides")
    tables = [torch.tensor([t.data_ptr() for t in ts], dtype=torch.int64, device=path.device)
              for ts in (k_trees, v_trees, k_caches, v_caches)]
    return _n.prepare_commit(k_trees[0], v_trees[0], k_caches[0], v_caches[0], None, path, accept_len, prefix_len, advance, n,
                             *tables, list(k_trees), list(v_trees), list(k_caches), list(v_caches))


def _paged_desc(q, k_pool, k_tree, out, scale):
    d = _make_desc(q, None, k_tree, out, scale)
    d.kc_stride_b, d.kc_stride_l, d.kc_stride_h = 0, k_pool.stride(1), k_pool.stride(2)
    return d


def prepare_tree_verify_attention_paged(q, k_pool, v_pool, block_table, k_tree, v_tree, parent, prefix_len, out,
                                        workspace, max_prefix_len: int, scale: float = 0.0) -> "PreparedCall":
    """jk_tree_verify_attention_paged with out and workspace given; nothing is launched.  k_pool, v_pool
    [n_pages, page_size, Hkv, D] (same strides), block_table int32 [B, max_blocks]."""
    return _n.prepare_attention(q, k_pool, v_pool, block_table, k_tree, v_tree, parent, prefix_len, int(max_prefix_len), scale, out,
                                workspace)


def tree_verify_attention_paged(q, k_pool, v_pool, block_table, k_tree, v_tree, parent, prefix_len,
                                max_prefix_len: int, scale: float = 0.0, out=None, workspace=None, stream=None):
    """jk_tree_verify_attention_paged; returns out [B,T,Hq,D] (allocated unless given)."""
    if workspace is None:
        d = _paged_desc(q, k_pool, k_tree, q if out is None else out, scale)
        need = int(lib().jk_tree_verify_attention_workspace(ctypes.byref(d), int(max_prefix_len)))
        if need == 0:
            raise JakiroError(3, "jk_tree_verify_attention_workspace")
        workspace = _new_workspace(need, q.device, stream)
    return _n.attention(q, k_pool, v_pool, block_table, k_tree, v_tree, parent, prefix_len, int(max_prefix_len), scale, out, workspace,
                        stream)


def prepare_commit_path_layers_paged(k_trees, v_trees, k_pools, v_pools, block_table, path, accept_len, prefix_len,
                                     advance: bool = True) -> "PreparedCall":
    """jk_commit_path_layers_paged for lists of per-layer tree tensors and page pools (one block table)."""
    import torch
    n = len(k_trees)
    for ts in (k_trees, v_trees, k_pools, v_pools):
        if len(ts) != n or any(t.stride() != ts[0].stride() or t.shape != ts[0].shape for t in ts):
            raise ValueError("per-layer tensors must share shape and strides")
    tables = [torch.tensor([t.data_ptr() for t in ts], dtype=torch.int64, device=path.device)
              for ts in (k_trees, v_trees, k_pools, v_pools)]
    return _n.prepare_commit(k_trees[0], v_trees[0], k_pools[0], v_pools[0], block_table, path, accept_len, prefix_len, advance, n,
                             *tables, list(k_trees), list(v_trees), list(k_pools), list(v_pools))


def prepare_accept_path(tree_tokens, parent, target_logits, mode, temperature, draft_probs, uniforms, out_path,
                        out_accept_len, out_bonus_token, workspace) -> "PreparedCall":
    """Same arguments as accept_path with outputs and workspace given; nothing is launched."""
    return _n.prepare_accept(tree_tokens, parent, target_logits, mode, temperature, draft_probs, None, uniforms, out_path,
                             out_accept_len, out_bonus_token, workspace)


def draft_heads_workspace(rows: int, d_model: int, vocab: int) -> int:
    return int(lib().jk_draft_heads_workspace(int(rows), int(d_model), int(vocab)))


def draft_heads(f_top, s_top, w_head, mode: int = JK_HEADS_DECOUPLED, temperature: float = 1.0, top_k: int = 10,
                alpha: float = 0.0, beta: float = 0.0, want_probs: bool = True, stream=None, out_probs=None):
    """jk_draft_heads.  f_top bf16 [R,2,d], s_top fp32 [R,2], w_head bf16 [V,d].
    Returns (logits [R,2,V], draft_probs [R,2,V] or None, topk_tokens [R,2,k] int32, topk_probs [R,2,k]).
    `out_probs` (contiguous fp32 [R,2,V], for instance rows of a round's table of draft distributions)
    receives the distributions instead of a new tensor."""
    return _n.draft_heads(f_top, s_top, w_head, mode, temperature, top_k, alpha, beta, want_probs, out_probs, stream)


def prepare_draft_heads(f_top, s_top, w_head, mode, temperature, top_k, alpha, beta, logits, draft_probs,
                        topk_tokens, topk_probs, workspace) -> "PreparedCall":
    """jk_draft_heads with outputs and workspace given; nothing is launched."""
    return _n.prepare_draft_heads(f_top, s_top, w_head, mode, temperature, top_k, alpha, beta, logits, draft_probs, topk_tokens,
                                  topk_probs, workspace)


def moe_experts_workspace(rows: int, d_model: int, d_ff: int, n_experts: int) -> int:
    return int(lib().jk_moe_experts_workspace(ctypes.byref(MoeDesc(int(rows), int(d_model), int(d_ff), int(n_experts)))))


def moe_experts(u, centroids, w_gate, w_up, w_down, want_mix: bool = True, stream=None):
    """jk_moe_experts.  Returns (f_top [R,2,d] bf16, s_top [R,2], expert_idx [R,2] int32, f_mix [R,d] bf16 or None)."""
    return _n.moe_experts(u, centroids, w_gate, w_up, w_down, want_mix, stream)


def prepare_moe_experts(u, centroids, w_gate, w_up, w_down, f_top, s_top, expert_idx, f_mix, workspace) -> "PreparedCall":
    """jk_moe_experts with outputs and workspace given; nothing is launched."""
    return _n.prepare_moe_experts(u, centroids, w_gate, w_up, w_down, f_top, s_top, expert_idx, f_mix, workspace)


class TreeState:
    """Device arrays of a growing draft tree (jk_tree_state), one set per batch."""

    def __init__(self, batch: int, max_nodes: int, device="cuda"):
        import torch
        self.batch, self.max_nodes = int(batch), int(max_nodes)
        self.tokens = torch.zeros((batch, max_nodes), dtype=torch.int32, device=device)
        self.parent = torch.full((batch, max_nodes), -1, dtype=torch.int32, device=device)
        self.score = torch.zeros((batch, max_nodes), dtype=torch.float32, device=device)
        self.q_row = torch.zeros((batch, max_nodes), dtype=torch.int32, device=device)
        self.n_nodes = torch.zeros((batch,), dtype=torch.int32, device=device)

    def reset(self) -> None:
        import torch
        # (a graph of torch.compile takes zero_, and no call of the extension)
        if torch.compiler.is_dynamo_compiling() or not _n.tree_reset(self.n_nodes):
            self.n_nodes.zero_()

    def desc(self) -> TreeStateDesc:
        return TreeStateDesc(_ptr(self.tokens), _ptr(self.parent), _ptr(self.score), _ptr(self.q_row),
                             _ptr(self.n_nodes), self.max_nodes)


def tree_grow(state: TreeState, frontier_in, cand_tokens, cand_probs, width: int, q_row_base: int, stream=None):
    """jk_tree_grow.  frontier_in int32 [B,n_front] or None (root); cand_tokens int32 / cand_probs fp32
    [B*n_front,2,k].  Returns the next frontier, int32 [B,width]."""
    return _n.tree_grow(state.tokens, state.parent, state.score, state.q_row, state.n_nodes, frontier_in, cand_tokens, cand_probs,
                        width, q_row_base, stream)


def tree_grow_tail(state: TreeState, frontier_in, cand_tokens, cand_probs, k1: int, k2: int, width: int,
                   q_row_base: int, stream=None) -> None:
    """jk_tree_grow_tail: children from head 0's lists, grandchildren from head 1's (contrastive mode)."""
    _n.tree_grow_tail(state.tokens, state.parent, state.score, state.q_row, state.n_nodes, frontier_in, cand_tokens, cand_probs, k1, k2,
                      width, q_row_base, stream)


def tree_fill_static(state: TreeState, frontier_in, cand_tokens, cand_probs, shape_slot, shape_expert, shape_rank,
                     next_index, q_row_base: int, stream=None):
    """jk_tree_fill_static.  shape_* int32 [n_new] device tensors; next_index int32 [n_next] or None.
    Returns (frontier_out int32 [B,n_next] or None, new_ids int32 [B,n_new])."""
    return _n.tree_fill_static(state.tokens, state.parent, state.score, state.q_row, state.n_nodes, frontier_in, cand_tokens,
                               cand_probs, shape_slot, shape_expert, shape_rank, next_index, q_row_base, stream)


def tree_finalize(state: TreeState, n_keep: int, stream=None):
    """jk_tree_finalize.  Returns (tree_tokens, parent, q_row, old_index) int32 [B,n_keep] and n_valid int32 [B]."""
    return _n.tree_finalize(state.tokens, state.parent, state.score, state.q_row, state.n_nodes, n_keep, stream)


def gather_draft_probs(q_all, q_row, stream=None):
    """jk_gather_draft_probs.  q_all fp32 [n_rows, V] (contiguous), q_row int32 [B, N] -> fp32 [B, N, V]."""
    return _n.gather_draft_probs(q_all, q_row, stream)


def linear(x, w, residual=None, out_dtype=None, stream=None):
    """jk_linear: x bf16 [m,k], w bf16 [n,k], residual bf16 [m,n] or None -> x @ w.T (+ residual) as bf16
    (default) or float32 (out_dtype=torch.float32)."""
    f32 = False
    if out_dtype is not None:
        import torch
        f32 = out_dtype == torch.float32
    return _n.linear(x, w, residual, f32, stream)


def accept_path_rows(tree_tokens, parent, target_logits, q_all, q_row, uniforms, temperature: float = 1.0,
                     max_depth: Optional[int] = None, workspace=None, stream=None):
    """jk_accept_path_rows (speculative sampling): like accept_path, with node k of sequence b tested against
    q_all[q_row[b, k]] (q_all fp32 [n_rows, V] contiguous, q_row int32 [B, N]) instead of a dense draft_probs."""
    if workspace is None:
        B, N = tree_tokens.shape
        workspace = _new_workspace(accept_path_workspace(B, N, target_logits.shape[-1], JK_SAMPLE), tree_tokens.device, stream)
    return _n.accept(tree_tokens, parent, target_logits, JK_SAMPLE, temperature, q_all, q_row, uniforms, max_depth, workspace, stream)
