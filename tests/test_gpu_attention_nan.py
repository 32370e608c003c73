"""A key whose score is no number, or +inf, makes the rows that see it NaN, and no others, however the key range is cut: whole,
in parts merged by a second launch or inside the kernel, of either data type."""
import numpy as np
import pytest
import torch

import paper_2502_06282_amd as jk
from workloads import CONFIGS, attention_inputs, round_to_bf16

from gpu_util import gpu_attention, oracle_attention, tune

pytestmark = pytest.mark.gpu

# (dtype, heads, KV heads, head_dim, nodes, prefix, knobs): fp32 whole, 8 parts, 16, 24 (a second launch); bf16 whole, two key
# columns, groups of 2 - 24 splits, pieces, 16 rows a workgroup
PATHS = {
    "f32_whole": ("f32", 4, 2, 64, 20, 200, {}), "f32_8": ("f32", 4, 2, 64, 20, 480, {}), "f32_8_launch": ("f32", 4, 2, 64, 20, 480, {"attn_fused": 0}),
    "f32_16": ("f32", 4, 4, 128, 20, 1400, {}), "f32_8_of_192": ("f32", 2, 2, 192, 20, 300, {}), "f32_24_of_192": ("f32", 2, 2, 192, 20, 2600, {}),
    "whole_4x1": ("bf16", 8, 2, 128, 60, 500, {"attn_wm": 4, "attn_wn": 1, "attn_splits": 1}),
    "whole_2x2": ("bf16", 8, 2, 64, 60, 500, {"attn_wm": 2, "attn_wn": 2, "attn_splits": 1}),
    "groups_4x1": ("bf16", 8, 2, 128, 60, 1500, {"attn_wm": 4, "attn_wn": 1, "attn_splits": 6, "attn_fused": 1}),
    "groups_of_2": ("bf16", 8, 2, 128, 60, 500, {"attn_wm": 4, "attn_wn": 1, "attn_splits": 2, "attn_fused": 1}),
    "groups_2x2": ("bf16", 8, 2, 64, 60, 1500, {"attn_wm": 2, "attn_wn": 2, "attn_splits": 3, "attn_fused": 1}),
    "groups_of_24": ("bf16", 8, 2, 128, 60, 3300, {"attn_wm": 4, "attn_wn": 1, "attn_splits": 24, "attn_fused": 1}),
    "launch": ("bf16", 8, 2, 128, 60, 1500, {"attn_wm": 4, "attn_wn": 1, "attn_splits": 6, "attn_fused": 0}),
    "launch_fine": ("bf16", 8, 2, 64, 60, 500, {"attn_wm": 2, "attn_wn": 2, "attn_splits": 2, "attn_fused": 0}),
    "pieces": ("bf16", 8, 2, 128, 60, 1500, {"attn_wm": 8, "attn_wn": 1, "attn_splits": 3}),
    "direct": ("bf16", 8, 2, 128, 60, 500, {"attn_wm": 1, "attn_wn": 4}),
}


@pytest.mark.parametrize("where", ["tree_nan", "prefix_nan", "prefix_inf"])
@pytest.mark.parametrize("path", PATHS)
def test_a_score_that_is_no_number_reaches_its_rows(path, where):
    dtype, H, Hkv, D, T, L, knobs = PATHS[path]
    cfg = CONFIGS["c3_llama3_8b"].with_(batch=2, n_tree=T, n_q_heads=H, n_kv_heads=Hkv, head_dim=D, prefix_len=L)
    x = attention_inputs(cfg, seed=D + L, scale_mult=np.sqrt(float(D)))
    if dtype == "bf16":
        x = {k: round_to_bf16(v) for k, v in x.items()}
    x = {k: np.array(v) for k, v in x.items()}
    par = np.tile(np.array([-1] + [(i - 1) // 2 for i in range(1, T)], dtype=np.int32), (2, 1))
    lens = [L, L - 37]
    G = H // Hkv
    none = np.zeros((2, T, H), dtype=bool)  # rows that are no number
    ref_x = x
    if where == "tree_nan":  # node 2 and what is below it, KV head 1 of sequence 1
        x["k_tree"][1, 2, 1, 5] = np.nan
        for i in range(T):
            n = i
            while n > 2:
                n = par[1, n]
            none[1, i, G:2 * G] = n == 2
        ref_x = dict(x, k_tree=np.nan_to_num(x["k_tree"]))
    elif where == "prefix_nan":
        x["k_cache"][0, 100, 0, D - 1] = np.nan
        none[0, :, :G] = True
        ref_x = dict(x, k_cache=np.nan_to_num(x["k_cache"]))
    else:  # +inf or -inf by the query's sign; -inf is a weight of zero: those rows as without that key
        x["k_cache"][0, 100, 0, 3] = np.inf
        assert (x["q"][0, :, :G, 3] != 0).all()
        none[0, :, :G] = x["q"][0, :, :G, 3] > 0
        ref_x = dict(x, k_cache=np.where(np.isinf(x["k_cache"]), 0.0, x["k_cache"]))
    ref = oracle_attention(**ref_x, parent=par, prefix_len=lens)
    if where == "prefix_inf":
        without = dict(x, k_cache=np.delete(x["k_cache"], 100, axis=1), v_cache=np.delete(x["v_cache"], 100, axis=1))
        ref[0, :, :G] = oracle_attention(**without, parent=par, prefix_len=[n - 1 for n in lens])[0, :, :G]
    for k, v in knobs.items():
        tune(k, v)
    got = gpu_attention(x, par, lens, dtype, max_prefix_len=L)
    assert np.isnan(got[none]).all()
    assert np.isfinite(got[~none]).all()
    # fp32: sums of at most 2600 terms of order one, a few units of rounding; bf16: two roundings of 2^-8 and a partial result's
    tol = (1e-5 if dtype == "f32" else 2.0 ** -6) * max(1.0, np.abs(ref[~none]).max())
    assert np.abs(got - ref)[~none].max() <= tol
