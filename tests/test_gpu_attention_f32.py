"""fp32 attention at the edges of what its waves ask for before the prefix length is known, against the fp64 oracle: lengths below
the bound, with values behind them that are no numbers, blocks that become shorter or are no more, undivided and divided ranges,
and trees of one to eight blocks beside them."""
import numpy as np
import pytest
import torch

import paper_2502_06282_amd as jk
from workloads import CONFIGS, attention_inputs

from gpu_util import gpu_attention, oracle_attention, to_dev, tune

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [32, 64, 80, 128, 192])
@pytest.mark.parametrize("bound,T", [(0, 1), (1, 17), (16, 16), (33, 64), (128, 10), (130, 128), (250, 33), (700, 20)])
def test_lengths_below_the_bound(D, bound, T):
    lens = [bound, bound // 2, 0, max(bound - 1, 0), min(15, bound), min(16, bound), min(17, bound), bound // 3]
    cfg = CONFIGS["c1_tiny"].with_(batch=len(lens), n_tree=T, n_q_heads=6, n_kv_heads=2, head_dim=D, prefix_len=bound)
    x = attention_inputs(cfg, seed=D + bound)
    rng = np.random.default_rng(T)
    par = np.stack([np.array([-1] + [int(rng.integers(-1, i)) for i in range(1, T)], dtype=np.int32) for _ in lens])
    ref = oracle_attention(**x, parent=par, prefix_len=lens)
    for b, n in enumerate(lens):
        x["k_cache"][b, n:] = np.nan
        x["v_cache"][b, n:] = np.nan
    got = gpu_attention(x, par, lens, "f32", max_prefix_len=bound)
    assert np.isfinite(got).all()
    # (sums of at most 830 fp32 terms of order one, a few units of rounding each: far below 1e-5 of the largest result)
    assert np.abs(got - ref).max() <= 1e-5 * max(1.0, np.abs(ref).max())


# keys of a bound whose ranges are 2, 3, 4, 5, 6, 8, 14 and 16 parts, and more than the kernel merges (24, and 10 and 16 of 192: a launch of
# its own), at lengths that leave parts empty
@pytest.mark.parametrize("B,H,D,T,bound", [(8, 8, 64, 20, 500), (5, 8, 128, 20, 300), (1, 8, 80, 17, 190), (1, 4, 256, 40, 100), (2, 4, 192, 20, 280), (1, 5, 132, 33, 400), (1, 3, 192, 20, 1800), (2, 3, 96, 33, 250),
                                           (2, 2, 16, 64, 450), (1, 6, 40, 50, 1900), (3, 2, 128, 1, 1500), (1, 3, 192, 20, 2600), (4, 3, 64, 64, 480),
                                           (1, 17, 64, 10, 1500), (1, 24, 192, 10, 1090)])
def test_parts_merged_by_the_last_workgroup(B, H, D, T, bound):
    """The same as merging them in a second launch, captured and replayed in a workspace whose partial results are
    noise each time; its words are zero again behind every call."""
    cfg = CONFIGS["c1_tiny"].with_(batch=B, n_tree=T, n_q_heads=H, n_kv_heads=H, head_dim=D, prefix_len=bound)
    x = attention_inputs(cfg, seed=bound)
    par = np.tile(np.array([-1] + [i // 2 for i in range(T - 1)], dtype=np.int32), (B, 1))
    lens = [(bound, 1, bound // 2, 0, bound - 1)[b % 5] for b in range(B)]
    ref = oracle_attention(**x, parent=par, prefix_len=lens)
    d = to_dev(x, "f32")
    parent, pl = torch.from_numpy(par).cuda(), torch.tensor(lens, dtype=torch.int32).cuda()
    ws = torch.zeros(jk.tree_verify_attention_workspace(d["q"], d["k_cache"], d["k_tree"], bound), dtype=torch.uint8, device="cuda")
    outs = {}
    for fused in (0, -1):
        tune("attn_fused", fused)
        out = torch.empty_like(d["q"])
        call = jk.prepare_tree_verify_attention(d["q"], d["k_cache"], d["v_cache"], d["k_tree"], d["v_tree"], parent, pl, out, ws,
                                                max_prefix_len=bound)
        call.launch()
        torch.cuda.synchronize()
        outs[fused] = out.clone()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
            call.launch()
        for rep in range(3):
            out.fill_(float("nan"))
            ws[jk.JK_WORKSPACE_HEADER_BYTES:].random_(0, 255)
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, outs[fused]), (fused, rep)
            assert not ws[:jk.JK_WORKSPACE_HEADER_BYTES].any()
    # (sums of at most 2600 fp32 terms of order one, as above; the two merges weigh the same parts and add them in another order)
    tol = 1e-5 * max(1.0, np.abs(ref).max())
    for out in outs.values():
        assert np.abs(out.double().cpu().numpy() - ref).max() <= tol
    assert (outs[0] - outs[-1]).abs().max().item() <= 1e-6 * max(1.0, np.abs(ref).max())
