"""fp32 attention at the edges of what its waves ask for before the prefix length is known, against the fp64 oracle: lengths below
the bound, with values behind them that are no numbers, blocks that become shorter or are no more, undivided and divided ranges,
and trees of one to eight blocks beside them."""
import numpy as np
import pytest

from workloads import CONFIGS, attention_inputs

from gpu_util import gpu_attention, oracle_attention

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
