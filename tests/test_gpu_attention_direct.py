"""The attention kernel of 16 query rows per workgroup that takes K and V straight into registers (csrc/tva_direct.hip) at its
edges, against the fp64 oracle: rows around a workgroup, keys around a block of 32 and a turn of the four waves, lengths below the
bound, paged caches beyond a lane's worth of page ids, scores that move the reference; and which calls the plan gives it."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2502_06282_amd as jk
from paper_2502_06282_amd import binding
from workloads import CONFIGS, attention_inputs, round_to_bf16

from gpu_util import check_attention, gpu_attention, oracle_attention, to_dev, tune

gpu = pytest.mark.gpu

# Unscaled inputs: outputs are of order 1/sqrt(keys) up to a few units.  Roundings: the weights' (2^-8, in numerator and
# denominator alike) and the result's (2^-8).  Relative to max|out| that is 2 * 2^-8 at most.
REL = 2.0 ** -7


def direct():
    tune("attn_wm", 1); tune("attn_wn", 4)


def _cfg(T, G, Hkv, D, L, B=1):
    return CONFIGS["c3_llama3_8b"].with_(batch=B, n_tree=T, n_q_heads=G * Hkv, n_kv_heads=Hkv, head_dim=D, prefix_len=L)


def _tree(B, T, seed):
    rng = np.random.default_rng(seed)
    return np.stack([np.array([-1] + [int(rng.integers(-1, i)) for i in range(1, T)], dtype=np.int32) for _ in range(B)])


def _check(cfg, lens, seed=0):
    x = attention_inputs(cfg, seed=seed, scale_mult=np.sqrt(float(cfg.head_dim)))
    par = _tree(cfg.batch, cfg.n_tree, seed + 1)
    ref = oracle_attention(**x, parent=par, prefix_len=lens)
    for b, n in enumerate(lens):  # what lies behind a sequence's length must not be used
        x["k_cache"][b, n:] = np.nan
        x["v_cache"][b, n:] = np.nan
    direct()
    got = gpu_attention(x, par, lens, "bf16", max_prefix_len=cfg.prefix_len)
    assert np.isfinite(got).all()
    assert np.abs(got - ref).max() <= REL * np.abs(ref).max()
    return got


@gpu
@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("T,G,L", [(1, 1, 5), (15, 1, 40), (16, 1, 300), (17, 1, 97), (3, 5, 64), (65, 1, 130), (64, 4, 31), (127, 2, 33), (128, 8, 200)])
def test_rows(D, T, G, L):
    _check(_cfg(T, G, 2, D, L), [L], seed=T * G)


@gpu
@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("L", [0, 1, 31, 32, 33, 96, 97, 127, 128, 129, 160, 256, 257, 700])
def test_prefixes(D, L):
    """Ends in every wave's first and later blocks; trees of one, two and four blocks behind them."""
    for T in (1, 32, 33, 128):
        _check(_cfg(T, 2, 1, D, max(L, 1)), [L], seed=L + T)


@gpu
@pytest.mark.parametrize("D", [128, 64])
def test_lengths_below_the_bound(D):
    """Blocks that were asked for on the assumed length and stay, are cut short, become the tree's, or are no more."""
    _check(_cfg(40, 4, 3, D, 300, 12), [300, 299, 0, 1, 31, 32, 63, 64, 128, 129, 160, 225], seed=D)


@gpu
@pytest.mark.parametrize("page,L", [(32, 500), (96, 300), (32, 8900)])
def test_paged_equals_contiguous(page, L):
    """Bit by bit, pages in any order, poison in front of, between and behind them; more blocks than a wave holds page ids for."""
    cfg, lens = _cfg(20, 4, 2, 128, L, 3), [L, 1, L // 2]
    x, par = attention_inputs(cfg, seed=page), _tree(3, 20, page)
    direct()
    want = gpu_attention(x, par, lens, "bf16")
    d, nb = to_dev(x, "bf16"), -(-L // page)
    table = torch.randperm(3 * nb + 2, device="cuda", generator=torch.Generator("cuda").manual_seed(page))[:3 * nb].reshape(3, nb).to(torch.int32).contiguous()
    kp = torch.full((3 * nb + 2, page, 2, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
    vp = kp.clone()
    for b, n in enumerate(lens):
        for j in range(-(-n // page)):
            m = min(page, n - j * page)
            kp[table[b, j], :m] = d["k_cache"][b, j * page:j * page + m]
            vp[table[b, j], :m] = d["v_cache"][b, j * page:j * page + m]
        table[b, -(-n // page):] = 10 ** 6 * (-1) ** b  # (entries behind the length may hold anything)
    ws = torch.empty(jk.tree_verify_attention_workspace(d["q"], None, d["k_tree"], L), dtype=torch.uint8, device="cuda")
    jk.workspace_init(ws)

    def call():
        return jk.tree_verify_attention_paged(d["q"], kp, vp, table, d["k_tree"], d["v_tree"], torch.from_numpy(par).cuda(),
                                              torch.tensor(lens, dtype=torch.int32, device="cuda"), L, workspace=ws).float().cpu().numpy()

    np.testing.assert_array_equal(call(), want)
    assert jk.last_device_error(ws) == 0
    table[2, 0] = 3 * nb + 2  # an id outside the pool that a result depends on
    call()
    assert jk.last_device_error(ws) == jk.JK_DEVERR_BAD_PAGE


@gpu
@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("where", [2, 40, 299, 510])
def test_outlier_key(D, where):
    """A score some hundred binary orders above the others, in a wave's first, second or last block."""
    cfg = _cfg(40, 4, 2, D, 520)
    x, par = attention_inputs(cfg, seed=where, scale_mult=np.sqrt(float(D))), _tree(1, 40, 3)
    x["k_cache"][0, where, 0] = round_to_bf16(12.0 * x["q"][0, 3, 1])
    direct()
    # (a one-hot row returns a value row, entries up to 4.5: two roundings of that)
    got, _ = check_attention(x, par, [520], "bf16", 2 * 2.0 ** -8 * 4.5, rel_tol=REL)
    v = x["v_cache"][0, where, 0].astype(np.float64)
    assert np.abs(got[0, 3, 1] - v).max() <= 2.0 ** -7 * np.abs(v).max() + 1e-6


@gpu
def test_planned_call_in_other_layouts_and_with_a_bad_parent():
    """Head-major caches, strided queries and results; an entry that is no parent counts as the root and is reported."""
    cfg, lens = _cfg(30, 4, 8, 128, 150, 3), [150, 149, 20]
    x, par = attention_inputs(cfg, scale_mult=np.sqrt(128.0)), _tree(3, 30, 5)
    d = to_dev(x, "bf16")
    plen = torch.tensor(lens, dtype=torch.int32, device="cuda")
    assert jk.tree_verify_attention_plan(d["q"], d["k_cache"], d["k_tree"], 150)["wm"] == 1
    kc, vc = (t.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3) for t in (d["k_cache"], d["v_cache"]))
    q = torch.empty((3, 30, 2, 32, 128), dtype=torch.bfloat16, device="cuda")[:, :, 1]
    q.copy_(d["q"])
    out = torch.full((3, 30, 3, 32, 128), 7.0, dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(jk.tree_verify_attention_workspace(q, kc, d["k_tree"], 150), dtype=torch.uint8, device="cuda")
    jk.workspace_init(ws)
    bad = par.copy()
    bad[1, 4], bad[2, 29] = 4, -2
    par[1, 4], par[2, 29] = -1, -1
    ref = oracle_attention(**x, parent=par, prefix_len=lens)
    for tree, err in ((par, 0), (bad, jk.JK_DEVERR_BAD_TREE)):
        out.fill_(7.0)
        got = jk.tree_verify_attention(q, kc, vc, d["k_tree"], d["v_tree"], torch.from_numpy(tree).cuda(), plen, max_prefix_len=150,
                                       out=out[:, :, 1], workspace=ws).float().cpu().numpy()
        assert np.abs(got - ref).max() <= REL * np.abs(ref).max()
        assert (out[:, :, 0] == 7).all() and (out[:, :, 2] == 7).all()
        assert jk.last_device_error(ws) == err


def test_which_calls_the_plan_gives_it():
    """Host only: calls of few keys, in one piece and with no room for partial results; never those beyond the line's range."""
    lib = binding.lib()

    def plan(B, T, G, Hkv, D, L):
        Hq = G * Hkv
        d = binding.AttnDesc(B, T, Hq, Hkv, D, T * Hq * D, Hq * D, D, Hkv * D, Hkv * D, D, T * Hkv * D, Hkv * D, D, T * Hq * D, Hq * D, D, 0.0, 0)
        out = (ctypes.c_int32 * 6)()
        assert lib.jk_tree_verify_attention_plan(ctypes.byref(d), L, out) == 0
        return list(out)

    for D in (64, 128):
        for B, T, G, Hkv, L in ((1, 10, 4, 8, 128), (1, 60, 4, 8, 64), (8, 5, 4, 8, 100), (2, 1, 8, 2, 33)):
            assert plan(B, T, G, Hkv, D, L) == [1, 4, 1, -(-T * G // 16), 1, 0]
        for B, T, G, Hkv, L in ((1, 60, 4, 8, 4096), (16, 60, 4, 8, 512), (1, 2, 1, 8, 1000)):
            assert plan(B, T, G, Hkv, D, L)[0] != 1


@pytest.mark.parametrize("splits", [0, 2, 64])
@pytest.mark.parametrize("L", [0, 300, 40000, 2000000])
def test_the_forced_kernel_takes_every_range(splits, L):
    """Host only: it has no splits, whatever number is forced and however long the range that a plan can have."""
    lib = binding.lib()
    d = binding.AttnDesc(2, 20, 8, 2, 128, 20 * 1024, 1024, 128, 256, 256, 128, 20 * 256, 256, 128, 20 * 1024, 1024, 128, 0.0, 0)
    out = (ctypes.c_int32 * 6)()
    try:
        for name, v in ((b"attn_wm", 1), (b"attn_wn", 4), (b"attn_splits", splits)):
            lib.jk_set_tuning(name, v)
        assert lib.jk_tree_verify_attention_plan(ctypes.byref(d), L, out) == 0 and list(out) == [1, 4, 1, 5, 1, 0]
        assert lib.jk_tree_verify_attention_workspace(ctypes.byref(d), L) >= jk.JK_WORKSPACE_HEADER_BYTES
    finally:
        for name in (b"attn_wm", b"attn_wn", b"attn_splits"):
            lib.jk_set_tuning(name, 0)


@gpu
def test_the_forced_kernel_beyond_what_others_take_undivided():
    """More keys than a workgroup of the others has page ids for (1024 tiles), two splits asked for."""
    tune("attn_splits", 2)
    _check(_cfg(5, 2, 1, 64, 33000), [33000], seed=7)
