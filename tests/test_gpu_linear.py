"""GPU parity: jk_linear (through the C ABI) against x w^T (+ residual), and Eq. 1 assembled from library
calls (projections -> tree attention over the draft layer's cache -> output projection + residual)
against the oracle's draft_attention_block."""
import numpy as np
import pytest
import torch

import paper_2502_06282_amd as jk
from gpu_util import tune
from oracle import draft_head as dh
from workloads import round_to_bf16

pytestmark = pytest.mark.gpu


def _bf(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda().to(torch.bfloat16)


@pytest.mark.parametrize("m,n,k", [(1, 128, 128), (7, 300, 256), (33, 1000, 384), (80, 4096, 1024), (256, 513, 128),
                                   (10, 768, 4096)])
def test_exact_arithmetic_inputs_are_bit_exact(m, n, k):
    rng = np.random.default_rng(m + n)
    x = rng.integers(-2, 3, size=(m, k)).astype(np.float32)
    w = (rng.integers(-1, 2, size=(n, k)) * 0.125).astype(np.float32)
    r = rng.integers(-4, 5, size=(m, n)).astype(np.float32)
    got = jk.linear(_bf(x), _bf(w), out_dtype=torch.float32).cpu().numpy()
    np.testing.assert_array_equal(got.astype(np.float64), dh.linear(x, w))
    got = jk.linear(_bf(x), _bf(w), _bf(r), out_dtype=torch.float32).cpu().numpy()
    np.testing.assert_array_equal(got.astype(np.float64), dh.linear(x, w, r))
    got = jk.linear(_bf(x), _bf(w), _bf(r)).float().cpu().numpy()          # bf16 output: one rounding
    np.testing.assert_array_equal(got, round_to_bf16(dh.linear(x, w, r).astype(np.float32)))


@pytest.mark.parametrize("m,n,k", [(20, 40001, 128), (128, 33000, 384), (130, 70001, 128), (160, 70016, 384)])
def test_wide_strips_are_bit_exact(m, n, k):
    """Outputs so wide that strips of 256 or 384 columns save a turn of workgroups: whole and ragged last strips, rows
    stored in one and in several groups, half chunks of k."""
    rng = np.random.default_rng(n)
    x = rng.integers(-2, 3, size=(m, k)).astype(np.float32)
    w = (rng.integers(-1, 2, size=(n, k)) * 0.125).astype(np.float32)
    got = jk.linear(_bf(x), _bf(w), out_dtype=torch.float32).cpu().numpy()
    np.testing.assert_array_equal(got.astype(np.float64), dh.linear(x, w))


def test_random_inputs_within_fp32_accumulation_error():
    rng = np.random.default_rng(1)
    m, n, k = 40, 2000, 2048
    x = round_to_bf16(rng.standard_normal((m, k), dtype=np.float32))
    w = round_to_bf16(rng.standard_normal((n, k), dtype=np.float32) / np.float32(np.sqrt(k)))
    got = jk.linear(_bf(x), _bf(w), out_dtype=torch.float32).cpu().numpy()
    ref = dh.linear(x, w)
    bound = k * 2.0 ** -23 * (np.abs(x).astype(np.float64) @ np.abs(w).astype(np.float64).T)
    assert (np.abs(got - ref) <= bound).all()


def test_eq1_block_from_library_calls():
    rng = np.random.default_rng(2)
    T, L, H, Hkv, D = 12, 300, 4, 2, 64
    d = H * D
    parent = np.array([-1, 0, 0, 1, 1, 2, 3, 3, 5, 6, 8, 8], dtype=np.int32)
    sc = np.float32(1.0 / np.sqrt(d))
    h = round_to_bf16(rng.standard_normal((T, d), dtype=np.float32))
    wq, wo = (round_to_bf16(rng.standard_normal((d, d), dtype=np.float32) * sc) for _ in range(2))
    wk, wv = (round_to_bf16(rng.standard_normal((Hkv * D, d), dtype=np.float32) * sc) for _ in range(2))
    kc, vc = (round_to_bf16(rng.standard_normal((L, Hkv, D), dtype=np.float32)) for _ in range(2))
    ref = dh.draft_attention_block(h, wq, wk, wv, wo, kc, vc, parent, H, Hkv)
    hd = _bf(h)
    q = jk.linear(hd, _bf(wq)).reshape(1, T, H, D)
    kt = jk.linear(hd, _bf(wk)).reshape(1, T, Hkv, D)
    vt = jk.linear(hd, _bf(wv)).reshape(1, T, Hkv, D)
    attn = jk.tree_verify_attention(q, _bf(kc)[None], _bf(vc)[None], kt, vt, torch.from_numpy(parent)[None].cuda(),
                                    torch.tensor([L], dtype=torch.int32).cuda())
    u = jk.linear(attn.reshape(T, d), _bf(wo), hd, out_dtype=torch.float32)
    torch.cuda.synchronize()
    err = np.abs(u.cpu().numpy() - ref).max()
    assert err <= 2e-2 * np.abs(ref).max(), err


def test_argument_errors():
    x = torch.zeros((4, 256), dtype=torch.bfloat16, device="cuda")
    w = torch.zeros((8, 256), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(jk.JakiroError) as e:
        jk.linear(x[:, :192].contiguous(), w[:, :192].contiguous())
    assert e.value.status == 3
    with pytest.raises(jk.JakiroError) as e:
        jk.linear(torch.zeros((257, 256), dtype=torch.bfloat16, device="cuda"), w)
    assert e.value.status == 3
    torch.cuda.synchronize()


@pytest.mark.parametrize("m,n,k", [(1, 1, 128), (16, 127, 384), (17, 129, 640), (48, 4100, 1152), (65, 128, 8192), (97, 33, 896),
                                   (129, 255, 256), (160, 257, 1920), (176, 513, 128), (241, 300, 2176), (3, 40000, 128)])
def test_row_blocks_strips_and_k_parts_at_their_edges(m, n, k):
    """Every row-block count of the streaming product with strips that end early, half chunks of k, one and many k parts,
    and an output that is not aligned for vector stores: bit-exact on exact-arithmetic inputs."""
    rng = np.random.default_rng(m + n + k)
    x = rng.integers(-2, 3, size=(m, k)).astype(np.float32)
    w = (rng.integers(-1, 2, size=(n, k)) * 0.125).astype(np.float32)
    r = rng.integers(-4, 5, size=(m, n)).astype(np.float32)
    want = dh.linear(x, w, r)
    got = jk.linear(_bf(x), _bf(w), _bf(r), out_dtype=torch.float32).cpu().numpy()
    np.testing.assert_array_equal(got.astype(np.float64), want)
    both = torch.full((2, m * n + 1), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(jk.lib().jk_linear_workspace(m, n, k), dtype=torch.uint8, device="cuda")
    xd, wd, rd, out16 = _bf(x), _bf(w), _bf(r), torch.empty(m * n, dtype=torch.bfloat16, device="cuda")
    st = jk.lib().jk_linear(m, n, k, xd.data_ptr(), wd.data_ptr(), rd.data_ptr(), out16.data_ptr(), both[1].data_ptr() + 4,
                            ws.data_ptr(), ws.numel(), None)
    torch.cuda.synchronize()
    assert st == 0
    np.testing.assert_array_equal(both[1, 1:].cpu().numpy().reshape(m, n).astype(np.float64), want)
    np.testing.assert_array_equal(out16.float().cpu().numpy().reshape(m, n), round_to_bf16(want.astype(np.float32)))
    assert torch.isnan(both[0]).all() and torch.isnan(both[1, 0])


@pytest.mark.parametrize("m", [1, 8, 9, 16, 17, 40, 48, 49, 64, 65, 72, 81, 97, 113, 128])
@pytest.mark.parametrize("n,k", [
    (1, 128), (7, 384), (1025, 640), (2047, 1024), (2500, 1152),        # strips of 4 - 12 rows; waves without a share of k,
    (4096, 2048), (4100, 1664), (6144, 4096), (8190, 1024),             # with one, with an odd number of them
    (12288, 512), (16384, 1024), (16385, 512),                          # strips of 48 and 64 rows; one more than that
])
def test_few_columns_are_bit_exact(m, n, k):
    """Products for which a workgroup takes a strip of a few weight rows and all of k, and those just beyond; small whole
    numbers, so that every order of summation gives the same."""
    rng = np.random.default_rng(m + n + k)
    x = rng.integers(-2, 3, size=(m, k)).astype(np.float32)
    w = rng.integers(-1, 2, size=(n, k)).astype(np.float32) * np.float32(0.125)
    r = rng.integers(-4, 5, size=(m, n)).astype(np.float32)
    want = x @ w.T + r                                                    # (exact in fp32: multiples of 1/8 below 2^12)
    got = jk.linear(_bf(x), _bf(w), _bf(r), out_dtype=torch.float32).cpu().numpy()
    np.testing.assert_array_equal(got, want)
    np.testing.assert_array_equal(jk.linear(_bf(x), _bf(w), _bf(r)).float().cpu().numpy(), round_to_bf16(want))


def _exact_case(m, n, k, seed):
    rng = np.random.default_rng(seed)
    x = rng.integers(-2, 3, size=(m, k)).astype(np.float32)
    w = rng.integers(-1, 2, size=(n, k)).astype(np.float32) * np.float32(0.125)
    r = rng.integers(-4, 5, size=(m, n)).astype(np.float32)
    return x, w, r, x @ w.T + r                                           # (exact in fp32: multiples of 1/8 below 2^14)


@pytest.mark.parametrize("m,n,k", [(64, 4096, 4096), (41, 4096, 8192), (24, 4100, 8320), (57, 8191, 8192), (64, 2049, 8064), (33, 5120, 10240),
                                   (65, 4096, 4096), (128, 2048, 4096), (97, 4096, 8192), (73, 6141, 4096),   # X in two blocks, with and without parts of k,
                                   (80, 6760, 7296), (128, 7012, 2048), (65, 1028, 4096)])                    # and strips that the XCDs do not divide
def test_two_workgroups_per_strip_are_bit_exact(m, n, k):
    """Products whose k is cut in two: the second workgroup of a strip to finish adds up both.  The workspace may hold
    anything (its words are not cleared for the call), is used by several calls in turn, and nothing is written behind it."""
    x, w, r, want = _exact_case(m, n, k, m + n)
    xd, wd, rd = _bf(x), _bf(w), _bf(r)
    need = jk.lib().jk_linear_workspace(m, n, k)
    out = torch.empty((m, n), dtype=torch.float32, device="cuda")
    for fill in (0, 0xFF, 0x80):
        ws = torch.full((need + 256,), fill, dtype=torch.uint8, device="cuda")
        for _ in range(3):
            out.fill_(float("nan"))
            assert jk.lib().jk_linear(m, n, k, xd.data_ptr(), wd.data_ptr(), rd.data_ptr(), None, out.data_ptr(), ws.data_ptr(), need,
                                      torch.cuda.current_stream().cuda_stream) == 0
            np.testing.assert_array_equal(out.cpu().numpy(), want)
        assert (ws[need:] == fill).all()


def test_linear_layers_replay_in_a_graph():
    """A graph keeps the words of its launches' meetings: every replay gives the eager result, with eager calls on the same
    buffers between them."""
    x, w, r, want = _exact_case(48, 4096, 8192, 5)
    x2, w2, r2, want2 = _exact_case(64, 4096, 4096, 6)
    a = [_bf(v) for v in (x, w, r)], [_bf(v) for v in (x2, w2, r2)]
    for t in a:
        jk.linear(*t)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = [jk.linear(*t, out_dtype=torch.float32) for t in a for _ in range(2)]
    for _ in range(6):
        for g in got:
            g.fill_(float("nan"))
        graph.replay()
        eager = jk.linear(*a[0], out_dtype=torch.float32)
        torch.cuda.synchronize()
        for g, e in zip(got, (want, want, want2, want2)):
            np.testing.assert_array_equal(g.cpu().numpy(), e)
        np.testing.assert_array_equal(eager.cpu().numpy(), want)


@pytest.mark.parametrize("forced", [0, 1], ids=["strips", "few_columns"])
@pytest.mark.parametrize("m,n,k", [(1, 60, 384), (64, 4100, 1152), (80, 6760, 640), (128, 8192, 256)])
def test_either_kernel_takes_a_layer(forced, m, n, k):
    x, w, r, want = _exact_case(m, n, k, m + k)
    for force in (forced, -1, forced):                   # (a thread's last plan is that of the last call's knob)
        tune("narrow_gemm", force)
        np.testing.assert_array_equal(jk.linear(_bf(x), _bf(w), _bf(r), out_dtype=torch.float32).cpu().numpy(), want)
