"""Division by multiplication (csrc/jk_divide.h), on the host; and a call that needs more than 32 bits of it."""
import os
import subprocess

import numpy as np
import pytest
import torch

import paper_2502_06282_amd as jk

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2502_06282_amd", "csrc")


def test_division_by_multiplication_is_exact(tmp_path):
    exe = str(tmp_path / "divide")
    subprocess.run(["g++", "-O1", "-std=c++17", "-w", "-I", CSRC, os.path.join(HERE, "divide.cpp"), "-o", exe], check=True, timeout=120)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout[-4000:]


@pytest.mark.gpu
@pytest.mark.parametrize("L", [0, 40, 400])
def test_thousands_of_query_heads_to_a_kv_head(L):
    """fp32, 128 nodes of 8191 heads: rows times heads pass 2^32.  Keys of zeros: a result is the mean of the values its node
    sees, the same for every head (sums of at most 528 terms of order one: a few units of fp32 rounding)."""
    T, H, D = 128, 8191, 4
    g = torch.Generator().manual_seed(L)
    v_cache, v_tree = torch.randn((1, max(L, 1), 1, D), generator=g), torch.randn((1, T, 1, D), generator=g)
    par = np.array([[-1] + [i // 3 for i in range(T - 1)]], dtype=np.int32)
    want = torch.empty((T, D), dtype=torch.float64)
    for i in range(T):
        seen, n = [], i
        while n >= 0:
            seen.append(n)
            n = int(par[0, n])
        want[i] = torch.cat([v_cache[0, :L, 0], v_tree[0, seen, 0]]).double().mean(0)
    z = lambda *s: torch.zeros(s, device="cuda")  # noqa: E731
    out = jk.tree_verify_attention(torch.randn((1, T, H, D), generator=g).cuda(), z(1, max(L, 1), 1, D), v_cache.cuda(), z(1, T, 1, D),
                                   v_tree.cuda(), torch.from_numpy(par).cuda(), torch.tensor([L], dtype=torch.int32).cuda(), max_prefix_len=L)
    torch.cuda.synchronize()
    assert (out[0].double().cpu() - want[:, None]).abs().max().item() <= 1e-5
