"""The attention kernel of 256 query rows per workgroup (csrc/tva_wide.hip) at its edges, against the fp64 oracle: rows
around a block of 32, a wave of 64 and a workgroup; prefixes around a tile, a run of four tiles and the K/V ring; pieces
merged pairwise; batches dealt out by length; paged caches; the repeat of a piece whose scores leave the reference frame."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2502_06282_amd as jk
from paper_2502_06282_amd import binding
from workloads import CONFIGS, attention_inputs, round_to_bf16, tree_for_config

from gpu_util import check_attention, gpu_attention, oracle_attention, to_dev, tune

gpu = pytest.mark.gpu

# Unscaled inputs: outputs are of order 1/sqrt(keys) up to a few units.  Roundings: the weights' (2^-8, in numerator and
# denominator alike) and the result's (2^-8); partial results are fp32.  Relative to max|out| that is 2 * 2^-8 at most.
REL = 2.0 ** -7


def wide(splits):
    tune("attn_wm", 8); tune("attn_wn", 1); tune("attn_splits", splits)


def _cfg(T, G, Hkv, D, L, B=1):
    return CONFIGS["c3_llama3_8b"].with_(batch=B, n_tree=T, n_q_heads=G * Hkv, n_kv_heads=Hkv, head_dim=D, prefix_len=L)


def _tree(B, T, seed):
    rng = np.random.default_rng(seed)
    return np.stack([np.array([-1] + [int(rng.integers(-1, i)) for i in range(1, T)], dtype=np.int32) for _ in range(B)])


def _check(cfg, lens, seed=0):
    x = attention_inputs(cfg, seed=seed, scale_mult=np.sqrt(float(cfg.head_dim)))
    par = _tree(cfg.batch, cfg.n_tree, seed + 1)
    ref = oracle_attention(**x, parent=par, prefix_len=lens)
    got = gpu_attention(x, par, lens, "bf16", max_prefix_len=max(cfg.prefix_len, 1))
    assert np.isfinite(got).all()
    assert np.abs(got - ref).max() <= REL * np.abs(ref).max()
    return got


@gpu
@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("T,G", [(1, 1), (31, 1), (33, 1), (64, 1), (65, 1), (127, 2), (64, 4), (129 // 2, 8), (100, 8)])
def test_rows(D, T, G):
    wide(1)
    _check(_cfg(T, G, 2, D, 300), [300], seed=T * G)


@gpu
@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("L", [0, 1, 31, 32, 33, 4 * 32, 5 * 32, 5 * 32 + 1, 8 * 32, 9 * 32 - 1, 13 * 32, 16 * 32, 17 * 32 + 5, 21 * 32, 900, 1300])
def test_prefixes(D, L):
    """Ends in every place of a run of four tiles and of the ring; trees of one, two and four tiles behind them."""
    for T in (20, 60, 128):
        wide(1)
        _check(_cfg(T, 2, 1, D, max(L, 1)), [L], seed=L + T)


@gpu
@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("splits", [2, 3, 4, 5, 7, 8])
def test_pieces(D, splits):
    """Pieces without a mask, with only masked tiles, and of every place in a run of four; the same bits however often."""
    cfg = _cfg(100, 4, 2, D, 1030)
    wide(splits)
    outs = [_check(cfg, [L]) for L in (1030, 1024, 700)]
    for L, first in zip((1030, 1024, 700), outs):
        for _ in range(3):
            np.testing.assert_array_equal(_check(cfg, [L]), first)


@gpu
@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("splits", [2, 3, 5, 8])
def test_merge_when_the_wait_expires(D, splits):
    """spin_limit 0: nobody waits for the other one's stores, the later of two that have left their results adds them.  Same
    bits, the error word says that waits expired, and the workspace (its words are zero again) serves normal calls."""
    cfg = _cfg(100, 8, 8, D, 1500, 2)
    x, par = attention_inputs(cfg, scale_mult=np.sqrt(float(D))), _tree(2, 100, splits)
    d = to_dev(x, "bf16")
    parent, plen = torch.from_numpy(par).cuda(), torch.tensor([1500, 1490], dtype=torch.int32, device="cuda")
    wide(splits)
    ws = torch.empty(jk.tree_verify_attention_workspace(d["q"], d["k_cache"], d["k_tree"], 1500), dtype=torch.uint8, device="cuda")
    jk.workspace_init(ws)

    def call():
        out = jk.tree_verify_attention(d["q"], d["k_cache"], d["v_cache"], d["k_tree"], d["v_tree"], parent, plen, workspace=ws)
        torch.cuda.synchronize()
        assert not ws[256:jk.JK_WORKSPACE_HEADER_BYTES].any()
        return out

    ref = call()
    assert jk.last_device_error(ws) == 0
    tune("spin_limit", 0)
    for _ in range(5):
        assert torch.equal(call(), ref)
    # (of two pieces the one with the tree comes long after the other one's stores; of more, two of equal length meet)
    assert jk.last_device_error(ws) in ((0, jk.JK_DEVERR_MERGE_WAIT) if splits == 2 else (jk.JK_DEVERR_MERGE_WAIT,))
    tune("spin_limit", -1)
    jk.workspace_init(ws[:jk.JK_WORKSPACE_HEADER_BYTES])
    for _ in range(3):
        assert torch.equal(call(), ref)
    assert jk.last_device_error(ws) == 0


@gpu
@pytest.mark.parametrize("splits", [1, 2, 3, 6])
@pytest.mark.parametrize("lens", [[600, 3, 90], [0, 600, 599, 1, 64], [600] * 4, [600] + [7] * 63])
def test_batches(lens, splits):
    """Sequences dealt out by length: one much longer than the others, empty ones, all alike, as many as a wave has lanes."""
    wide(splits)
    B = len(lens)
    _check(_cfg(12 if B > 8 else 50, 8 if B > 8 else 4, 1 if B > 8 else 2, 128, 600, B), lens, seed=B + splits)


@gpu
def test_prefix_shorter_than_the_bound_and_more_than_64_sequences():
    wide(1)
    _check(_cfg(60, 4, 2, 128, 1000), [333])
    wide(2)
    _check(_cfg(60, 4, 2, 128, 1000), [999])
    cfg = _cfg(9, 12, 1, 64, 200, 70)
    _check(cfg, [200 - 2 * i for i in range(70)])


@gpu
@pytest.mark.parametrize("page", [32, 64, 128])
@pytest.mark.parametrize("splits", [1, 3])
def test_paged_equals_contiguous(page, splits):
    cfg = _cfg(70, 4, 2, 128, 1000, 3)
    lens = [1000, 130, 777]
    x, par = attention_inputs(cfg, seed=page), _tree(3, 70, page)
    wide(splits)
    want = gpu_attention(x, par, lens, "bf16")
    d, nb = to_dev(x, "bf16"), -(-1000 // page)
    table = torch.randperm(3 * nb + 2, device="cuda", generator=torch.Generator("cuda").manual_seed(page))[:3 * nb].reshape(3, nb).to(torch.int32).contiguous()
    kp = torch.full((3 * nb + 2, page, 2, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
    vp = kp.clone()
    for b, n in enumerate(lens):
        for j in range(-(-n // page)):
            m = min(page, n - j * page)
            kp[table[b, j], :m] = d["k_cache"][b, j * page:j * page + m]
            vp[table[b, j], :m] = d["v_cache"][b, j * page:j * page + m]
    got = jk.tree_verify_attention_paged(d["q"], kp, vp, table, d["k_tree"], d["v_tree"], torch.from_numpy(par).cuda(),
                                         torch.tensor(lens, dtype=torch.int32, device="cuda"), 1000)
    np.testing.assert_array_equal(got.float().cpu().numpy(), want)


@gpu
@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("splits", [1, 3])
@pytest.mark.parametrize("where", [5, 700, 1099])
def test_outlier_key(D, splits, where):
    """A score some hundred binary orders above everything in front of it: the piece is done once more."""
    wide(splits)
    cfg = _cfg(40, 4, 2, D, 1100)
    x, par = attention_inputs(cfg, seed=where, scale_mult=np.sqrt(float(D))), _tree(1, 40, 3)
    x["k_cache"][0, where, 0] = round_to_bf16(12.0 * x["q"][0, 3, 1])
    # (a one-hot row returns a value row, entries up to 4.5: two roundings of that)
    got, _ = check_attention(x, par, [1100], "bf16", 2 * 2.0 ** -8 * 4.5, rel_tol=REL)
    v = x["v_cache"][0, where, 0].astype(np.float64)
    assert np.abs(got[0, 3, 1] - v).max() <= 2.0 ** -7 * np.abs(v).max() + 1e-6


@gpu
def test_planned_calls_agree_with_the_other_kernels():
    """Calls the plan gives to this kernel, in other layouts as well: head-major caches, strided queries and results."""
    for cfg, lens in ((_cfg(100, 8, 8, 128, 8192, 4), [8192, 8000, 8191, 4000]), (_cfg(46, 4, 8, 64, 6000, 12), [6000 - 300 * i for i in range(12)])):
        x, par = attention_inputs(cfg, scale_mult=np.sqrt(float(cfg.head_dim))), _tree(cfg.batch, cfg.n_tree, 5)
        d = to_dev(x, "bf16")
        parent, plen = torch.from_numpy(par).cuda(), torch.tensor(lens, dtype=torch.int32, device="cuda")
        assert jk.tree_verify_attention_plan(d["q"], d["k_cache"], d["k_tree"], cfg.prefix_len)["wm"] == 8
        kc, vc = (t.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3) for t in (d["k_cache"], d["v_cache"]))
        q = torch.empty((*d["q"].shape[:2], 2, *d["q"].shape[2:]), dtype=torch.bfloat16, device="cuda")[:, :, 1]
        q.copy_(d["q"])
        out = torch.full_like(torch.empty((*q.shape[:2], 3, *q.shape[2:]), device="cuda"), 7.0, dtype=torch.bfloat16)
        a = jk.tree_verify_attention(q, kc, vc, d["k_tree"], d["v_tree"], parent, plen, max_prefix_len=cfg.prefix_len, out=out[:, :, 1])
        assert (out[:, :, 0] == 7).all() and (out[:, :, 2] == 7).all()
        tune("attn_wm", 4); tune("attn_wn", 1); tune("attn_splits", 1)
        b = jk.tree_verify_attention(d["q"], d["k_cache"], d["v_cache"], d["k_tree"], d["v_tree"], parent, plen)
        tune("attn_wm", 0); tune("attn_wn", 0); tune("attn_splits", 0)
        a, b = a.float(), b.float()
        assert float((a - b).abs().max()) <= 2 * REL * float(b.abs().max())


def test_workspace_covers_every_smaller_call():
    """Host only: the partial results of every plan this kernel gets fit the workspace that was sized for a larger call."""
    rng = np.random.default_rng(2)
    lib = binding.lib()

    def desc(B, T, Hq, Hkv, D):
        return binding.AttnDesc(B, T, Hq, Hkv, D, T * Hq * D, Hq * D, D, Hkv * D, Hkv * D, D, T * Hkv * D, Hkv * D, D, T * Hq * D, Hq * D, D, 0.0, 0)

    seen = 0
    for _ in range(1500):
        G, Hkv, D = int(rng.choice([1, 4, 8])), int(rng.choice([1, 2, 8, 32])), int(rng.choice([64, 128]))
        B, T, L = int(rng.integers(1, 33)), int(rng.integers(1, 129)), int(np.exp(rng.uniform(np.log(32), np.log(60000))))
        out = (ctypes.c_int32 * 6)()
        assert lib.jk_tree_verify_attention_plan(ctypes.byref(desc(B, T, G * Hkv, Hkv, D)), L, out) == 0
        if out[0] != 8:
            continue
        seen += 1
        need = 32768 + (B * Hkv * out[4] * out[3] * 256 * (4 * D + 8) if out[4] > 1 else 0)
        for big in ((B, T, L), (B + 3, T, L), (B, min(T + 9, 128), L), (B, T, 2 * L)):
            assert lib.jk_tree_verify_attention_workspace(ctypes.byref(desc(big[0], big[1], G * Hkv, Hkv, D)), big[2]) >= need
    assert seen > 50
