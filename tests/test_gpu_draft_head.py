"""GPU parity: jk_draft_heads (through the C ABI) against the draft-head oracle.

Logits: the library rounds the two head inputs to bf16 once (8 significant bits, round to nearest:
relative error at most 2^-8 per element) and accumulates products in fp32, so
|logit - oracle| <= (2^-8 + K 2^-23) * sum_k |x_k w_k| element by element.  The rounding errors are
independent and uniform within half a unit in the last place, i.e. of standard deviation at most
2^-7 / sqrt(12) relative to the element, so the root mean square of the logit errors must stay
below 2^-7 / sqrt(12) times the root mean square of sqrt(sum_k (x_k w_k)^2): a bound that a
systematic mistake sqrt(K) times smaller than the first one allows would still break.
Inputs whose products and sums are exact in fp32 must give the oracle's logits bit for bit.
Candidates are an integer decision taken on the library's own fp32 logits: they must equal the
oracle's selection applied to those logits exactly.  Probabilities: fp32 exp and a double
normaliser against the oracle's softmax of the same logits, relative 3e-5.
"""
import numpy as np
import pytest
import torch

import paper_2502_06282_amd as jk
from gpu_util import tune
from oracle import draft_head as dh
from workloads import draft_head_inputs

pytestmark = pytest.mark.gpu


def _call(x, mode=jk.JK_HEADS_DECOUPLED, temperature=1.0, top_k=5, alpha=0.0, beta=0.0, want_probs=True):
    f = torch.from_numpy(x["f_top"]).cuda().to(torch.bfloat16)
    s = torch.from_numpy(x["s_top"]).cuda()
    w = torch.from_numpy(x["w_head"]).cuda().to(torch.bfloat16)
    lg, q, tk, tp = jk.draft_heads(f, s, w, mode, temperature, top_k, alpha, beta, want_probs)
    torch.cuda.synchronize()
    return (lg.cpu().numpy(), None if q is None else q.cpu().numpy(), tk.cpu().numpy(), tp.cpu().numpy())


def _check(x, mode=jk.JK_HEADS_DECOUPLED, temperature=1.0, top_k=5, alpha=0.0, beta=0.0, exact=False):
    lg, q, tk, tp = _call(x, mode, temperature, top_k, alpha, beta)
    xin = dh.head_inputs(x["f_top"], x["s_top"], mode, alpha, beta)
    w = x["w_head"].astype(np.float64)
    ref = xin @ w.T
    K = w.shape[1]
    if exact:
        np.testing.assert_array_equal(lg.astype(np.float64), ref)
    else:
        bound = (2.0 ** -8 + K * 2.0 ** -23) * (np.abs(xin) @ np.abs(w).T) + 1e-30
        err = np.abs(lg - ref)
        assert (err <= bound).all(), f"worst ratio {np.max(err / bound):.3f}"
        spread = np.sqrt((xin * xin) @ (w * w).T)
        assert np.sqrt(np.mean(err ** 2)) <= 2.0 ** -7 / np.sqrt(12.0) * np.sqrt(np.mean(spread ** 2)) + 1e-30
    # decisions and probabilities from the library's own logits
    np.testing.assert_array_equal(tk, dh.top_candidates(lg, top_k))
    qref = dh.draft_distribution(lg, temperature)
    np.testing.assert_allclose(q, qref, rtol=3e-5, atol=1e-30)
    np.testing.assert_allclose(tp, np.take_along_axis(qref, tk.astype(np.int64), axis=-1), rtol=3e-5, atol=1e-30)
    return lg, q, tk, tp


def _exact_inputs(rows, d, vocab, seed):
    rng = np.random.default_rng(seed)
    return {"f_top": rng.integers(-2, 3, size=(rows, 2, d)).astype(np.float32),
            "s_top": np.stack([np.full(rows, 0.5), np.full(rows, 0.25)], 1).astype(np.float32),
            "w_head": (rng.integers(-1, 2, size=(vocab, d)) * 0.125).astype(np.float32)}


@pytest.mark.parametrize("rows,d,vocab", [(3, 256, 1000), (16, 128, 130), (17, 384, 4099), (128, 256, 513),
                                            (5, 1024, 3000), (40, 2048, 700), (90, 256, 600)])   # two of them split k
def test_exact_arithmetic_inputs_are_bit_exact(rows, d, vocab):
    _check(_exact_inputs(rows, d, vocab, rows), exact=True)
    _check(_exact_inputs(rows, d, vocab, rows + 1), mode=jk.JK_HEADS_CONTRASTIVE, alpha=0.5, beta=2.0, exact=True)


@pytest.mark.parametrize("rows", [1, 5, 16, 33, 40, 64, 80, 90, 100, 128])   # 1..8 row blocks of 32
def test_random_inputs_every_row_block_count(rows):
    _check(draft_head_inputs(rows, 512, 4096 + 37 * (rows % 4), seed=rows), top_k=10)


@pytest.mark.parametrize("rows,vocab,top_k", [(1, 1024, 16), (1, 1025, 2), (2, 5, 4), (1, 70003, 12), (66, 16388, 10),
                                              (66, 16385, 10), (70, 33001, 5), (70, 40000, 16)])
def test_rows_of_every_length(rows, vocab, top_k):
    """Rows from blocks' statistics, whole and cut into parts (by the number of rows and the vocabulary), rows that start at multiples of
    16 bytes and not, equal logits far from each other."""
    _check(draft_head_inputs(rows, 128, vocab, seed=vocab), top_k=top_k)
    _check(_exact_inputs(rows, 128, vocab, vocab), top_k=top_k, exact=True)


@pytest.mark.parametrize("forced,rows,vocab,top_k", [(1, 16, 33000, 16), (1, 2, 32772, 3), (1, 16, 49151, 11),              # 4 entries a thread
                                                     (-1, 33, 32769, 16), (-1, 40, 40000, 10), (-1, 60, 32772, 5),          # 8
                                                     (-1, 70, 33001, 5), (-1, 70, 40000, 16), (-1, 128, 32769, 12)])        # 16
def test_rows_cut_into_parts_of_every_length(forced, rows, vocab, top_k):
    """Calls whose product leaves no statistics (equal shares of the vocabulary, or more than 32 tokens), of rows too long to be taken whole:
    4, 8 and 16 entries a thread, whole and ragged last parts; then equal logits, more candidates than any list holds."""
    tune("ring_gemm", forced)
    _check(draft_head_inputs(rows, 128, vocab, seed=vocab), top_k=top_k)
    x = _exact_inputs(rows, 128, vocab, vocab)
    _check(x, top_k=top_k, temperature=0.8, exact=True)
    x["w_head"][:] = x["w_head"][0]
    lg, q, tk, tp = _check(x, top_k=top_k, exact=True)
    np.testing.assert_array_equal(tk, np.broadcast_to(np.arange(top_k), tk.shape))
    np.testing.assert_allclose(q, 1.0 / vocab, rtol=3e-5)


def test_widest_model_and_longest_candidate_lists():
    """d_model 16 384 and top-16, the largest the call takes (a small vocabulary keeps the oracle quick)."""
    _check(draft_head_inputs(3, 16384, 300, seed=5), top_k=16)
    _check(_exact_inputs(2, 16384, 257, 6), top_k=16, exact=True)


@pytest.mark.parametrize("mode,alpha,beta", [(jk.JK_HEADS_DECOUPLED, 0, 0), (jk.JK_HEADS_CONTRASTIVE, 0.3, 1.1),
                                             (jk.JK_HEADS_CONTRASTIVE, -0.25, 0.5)])
@pytest.mark.parametrize("temperature", [1.0, 0.6, 2.5])
def test_modes_and_temperatures(mode, alpha, beta, temperature):
    _check(draft_head_inputs(24, 1024, 32000, seed=11), mode, temperature, 10, alpha, beta)


def test_left_plus_right_is_the_mixture_head():
    x = _exact_inputs(8, 256, 777, 3)
    dec = _call(x)[0]
    con = _call(x, jk.JK_HEADS_CONTRASTIVE, alpha=1.0, beta=1.0)[0]
    np.testing.assert_array_equal(dec[:, 0] + dec[:, 1], con[:, 0])


def test_all_equal_logits_take_the_lowest_ids_and_a_uniform_distribution():
    x = draft_head_inputs(4, 256, 9000, seed=5)      # more ties than the candidate list holds
    x["f_top"][:, 1] = x["f_top"][:, 0]
    lg, q, tk, tp = _check(x, jk.JK_HEADS_CONTRASTIVE, alpha=0.75, beta=0.75, top_k=16)
    assert (lg[:, 1] == 0).all() and (tk[:, 1] == np.arange(16)).all()
    np.testing.assert_allclose(q[:, 1], 1.0 / 9000, rtol=1e-6)


def test_duplicated_embedding_rows_tie_towards_the_lower_id():
    # exact-arithmetic inputs: workgroups sum over k in different orders, so only sums without
    # rounding are guaranteed to agree bit for bit between the two copies of a row
    x = _exact_inputs(6, 256, 2048, 6)
    x["w_head"][1024:] = x["w_head"][:1024]
    lg, q, tk, tp = _check(x, top_k=8, exact=True)
    assert (lg[:, :, 1024:] == lg[:, :, :1024]).all()
    best = tk[:, :, 0]
    assert (best < 1024).all()        # of two equal logits the lower id comes first


def test_decoupled_heads_do_not_see_the_other_expert():
    x = draft_head_inputs(5, 256, 1500, seed=7)
    ref = _call(x)[0]
    x["f_top"][2, 1] = np.nan
    got = _call(x)[0]
    np.testing.assert_array_equal(got[:, 0], ref[:, 0])
    assert np.isnan(got[2, 1]).all() and np.isfinite(np.delete(got[:, 1], 2, axis=0)).all()


def test_probabilities_are_optional_and_rows_are_independent():
    x = draft_head_inputs(9, 256, 3000, seed=8)
    a = _call(x, top_k=4)
    b = _call(x, top_k=4, want_probs=False)
    assert b[1] is None
    np.testing.assert_array_equal(a[0], b[0])
    np.testing.assert_array_equal(a[2], b[2])
    np.testing.assert_array_equal(a[3], b[3])
    sub = {"f_top": x["f_top"][3:4], "s_top": x["s_top"][3:4], "w_head": x["w_head"]}
    np.testing.assert_array_equal(_call(sub, top_k=4)[0][0], a[0][3])


def test_argument_errors():
    x = draft_head_inputs(2, 256, 300, seed=9)
    f = torch.from_numpy(x["f_top"]).cuda().to(torch.bfloat16)
    s = torch.from_numpy(x["s_top"]).cuda()
    w = torch.from_numpy(x["w_head"]).cuda().to(torch.bfloat16)
    for kw, status in [(dict(temperature=0.0), 1), (dict(top_k=17), 3), (dict(top_k=0), 1), (dict(top_k=301), 1),
                       (dict(mode=2), 1), (dict(mode=1, alpha=float("nan")), 1)]:
        with pytest.raises(jk.JakiroError) as e:
            jk.draft_heads(f, s, w, **kw)
        assert e.value.status == status, kw
    with pytest.raises(jk.JakiroError) as e:       # d_model not a multiple of 128
        jk.draft_heads(f[:, :, :192].contiguous(), s, w[:, :192].contiguous())
    assert e.value.status == 3
    f129 = torch.zeros((129, 2, 256), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(jk.JakiroError) as e:
        jk.draft_heads(f129, torch.zeros((129, 2), device="cuda"), w)
    assert e.value.status == 3
    # workspace too small / missing
    R, d, V = 2, 256, 300
    lg = torch.empty((R, 2, V), device="cuda")
    tk = torch.empty((R, 2, 3), dtype=torch.int32, device="cuda")
    tp = torch.empty((R, 2, 3), device="cuda")
    small = torch.empty(256, dtype=torch.uint8, device="cuda")
    with pytest.raises(jk.JakiroError) as e:
        jk.prepare_draft_heads(f, s, w, 0, 1.0, 3, 0.0, 0.0, lg, None, tk, tp, small).launch()
    assert e.value.status == 4
    torch.cuda.synchronize()


def test_full_size_llama3_shape_sampled_against_the_oracle():
    """The shape the benchmark times: 80 hidden states (8 sequences x 10 expanded nodes), d = 4096, the
    128 256-token vocabulary.  Logits against the oracle on sampled vocabulary rows (including both
    ends of the last, ragged 128-row strip); candidates and probabilities on every row."""
    R, d, V, k = 80, 4096, 128256, 10
    x = draft_head_inputs(R, d, V, seed=12)
    lg, q, tk, tp = _call(x, temperature=1.0, top_k=k)
    rng = np.random.default_rng(0)
    ids = np.unique(np.concatenate([rng.integers(0, V, 1500), np.arange(0, 130), np.arange(V - 130, V)]))
    xin = dh.head_inputs(x["f_top"], x["s_top"], dh.DECOUPLED)
    w = x["w_head"][ids].astype(np.float64)
    ref = xin @ w.T
    bound = (2.0 ** -8 + d * 2.0 ** -23) * (np.abs(xin) @ np.abs(w).T)
    err = np.abs(lg[:, :, ids] - ref)
    assert (err <= bound).all()
    spread = np.sqrt((xin * xin) @ (w * w).T)
    assert np.sqrt(np.mean(err ** 2)) <= 2.0 ** -7 / np.sqrt(12.0) * np.sqrt(np.mean(spread ** 2))
    np.testing.assert_array_equal(tk, dh.top_candidates(lg, k))
    qref = dh.draft_distribution(lg, 1.0)
    np.testing.assert_allclose(q, qref, rtol=3e-5, atol=1e-30)
    np.testing.assert_allclose(tp, np.take_along_axis(qref, tk.astype(np.int64), axis=-1), rtol=3e-5)


def test_rows_with_fewer_finite_logits_than_candidates():
    """Only three tokens of the vocabulary have logits above -inf (the other embedding rows carry -inf against a
    positive feature): they come first, best first, with probabilities that sum to one; the remaining places of the
    candidate lists report token 0 with probability 0, and every other draft probability is an exact zero."""
    rows, d, V, k = 3, 256, 1500, 6
    x = draft_head_inputs(rows, d, V, seed=21)
    x["f_top"] = np.abs(x["f_top"]).astype(np.float32) + 0.5       # positive features
    x["s_top"] = np.full((rows, 2), 0.5, dtype=np.float32)
    w = x["w_head"].copy()
    alive = [7, 900, 1499]
    for v in range(V):
        if v not in alive:
            w[v] = 0.0
            w[v, 0] = -np.inf
    x["w_head"] = w
    lg, q, tk, tp = _call(x, top_k=k)
    dead = np.setdiff1d(np.arange(V), alive)
    assert np.isneginf(lg[:, :, dead]).all() and np.isfinite(lg[:, :, alive]).all()
    assert (q[:, :, dead] == 0).all()
    np.testing.assert_allclose(q[:, :, alive].sum(-1), 1.0, rtol=1e-6)
    for r in range(rows):
        for h in range(2):
            order = sorted(alive, key=lambda v: (-lg[r, h, v], v))
            assert tk[r, h, :3].tolist() == order
            np.testing.assert_allclose(tp[r, h, :3], q[r, h, order], rtol=1e-6)
            assert (tk[r, h, 3:] == 0).all() and (tp[r, h, 3:] == 0).all()


@pytest.mark.parametrize("rows", [1, 8, 9, 16, 17])      # one and two row blocks of 16 mixed by the product itself; one more
@pytest.mark.parametrize("d,vocab", [(128, 257), (640, 1025), (2048, 300), (384, 40000)])   # half chunks of k, divided k, whole k
def test_rows_mixed_by_the_product_are_bit_exact(rows, d, vocab):
    x = _exact_inputs(rows, d, vocab, rows + d)
    _check(x, exact=True)
    _check(x, mode=jk.JK_HEADS_CONTRASTIVE, alpha=0.5, beta=2.0, exact=True)
    x["f_top"][0, 1, 3] = np.nan                         # left out where its coefficient is zero
    lg, *_ = _call(x, mode=jk.JK_HEADS_CONTRASTIVE, alpha=0.0, beta=2.0)
    assert np.isnan(lg[0, 0]).all() and np.isfinite(lg[0, 1]).all() and np.isfinite(lg[1:]).all()


@pytest.mark.parametrize("rows", [18, 24, 25, 31, 32, 33])   # three and four row blocks of 16 mixed by the product; one more
@pytest.mark.parametrize("d,vocab", [(640, 1025), (2048, 300), (384, 70003)])
def test_more_rows_mixed_by_the_product_are_bit_exact(rows, d, vocab):
    test_rows_mixed_by_the_product_are_bit_exact(rows, d, vocab)
    x = _exact_inputs(rows, d, vocab, rows)
    x["f_top"][rows - 1, 0, 5] = np.inf                  # and here the row's own feature, the last row's
    lg, *_ = _call(x, mode=jk.JK_HEADS_CONTRASTIVE, alpha=0.5, beta=0.0)
    assert np.isfinite(lg[:-1]).all() and np.isfinite(lg[-1, 1]).all() and not np.isfinite(lg[-1, 0]).any()


@pytest.mark.parametrize("rows", [1, 4, 5, 12, 16])      # groups of eight rows, whole and not
@pytest.mark.parametrize("d,vocab", [(128, 8192), (640, 9001), (384, 16388), (256, 33003)])
def test_equal_shares_of_the_vocabulary_are_bit_exact(rows, d, vocab):
    """Vocabularies that strips of 128 rows would not fill the CUs with: batches of two, four and six groups of weight
    rows, the last ones short, waves without a share of k, odd row lengths."""
    x = _exact_inputs(rows, d, vocab, rows + d)
    _check(x, exact=True)
    _check(x, mode=jk.JK_HEADS_CONTRASTIVE, alpha=0.5, beta=2.0, exact=True)
    x["f_top"][0, 1, 3] = np.nan                         # left out where its coefficient is zero
    lg, *_ = _call(x, mode=jk.JK_HEADS_CONTRASTIVE, alpha=0.0, beta=2.0)
    assert np.isnan(lg[0, 0]).all() and np.isfinite(lg[0, 1]).all() and np.isfinite(lg[1:]).all()


@pytest.mark.parametrize("forced", [0, 1], ids=["strips", "equal_shares"])
@pytest.mark.parametrize("rows,d,vocab", [(1, 128, 700), (5, 640, 9001), (9, 512, 25752), (16, 384, 32768), (12, 256, 24577)])
def test_either_kernel_takes_the_heads(forced, rows, d, vocab):
    tune("ring_gemm", forced)
    test_equal_shares_of_the_vocabulary_are_bit_exact(rows, d, vocab)


@pytest.mark.parametrize("rows,d,vocab", [(1, 128, 5), (3, 128, 4096), (2, 128, 4097), (9, 4096, 300), (5, 128, 8192), (3, 128, 8193), (4, 1024, 12290),
                                          (1, 128, 12288), (2, 128, 16383), (33, 128, 16384), (31, 128, 16385), (32, 128, 16385), (32, 128, 20481),
                                          (33, 128, 24576), (32, 128, 28700), (34, 128, 32768), (32, 128, 32769), (33, 128, 5), (33, 128, 4096), (40, 128, 4097),
                                          (33, 128, 8193), (40, 128, 12290), (33, 128, 16385), (64, 128, 20481), (33, 128, 28672), (33, 128, 28673), (40, 128, 32767)])
def test_short_rows(rows, d, vocab):
    """Of more than 32 tokens, short rows are taken whole: the edges of what a thread holds, and the most that a workgroup takes.  Of fewer
    the same lengths from blocks' statistics.  Then rows of equal logits, all of them candidates (exact sums: 1 / vocab within
    the tolerance of every probability here)."""
    top_k = min(vocab, 11)
    x = _exact_inputs(rows, d, vocab, vocab)
    _check(x, top_k=top_k, temperature=0.8, exact=True)
    _check(draft_head_inputs(rows, d, vocab, seed=rows), top_k=top_k)
    x["w_head"][:] = x["w_head"][0]
    lg, q, tk, tp = _check(x, top_k=top_k, exact=True)
    np.testing.assert_array_equal(tk, np.broadcast_to(np.arange(top_k), tk.shape))
    np.testing.assert_allclose(q, 1.0 / vocab, rtol=3e-5)


@pytest.mark.parametrize("vocab", [5, 127, 128, 129, 1001, 16385, 33000, 131072, 140003])
@pytest.mark.parametrize("rows", [1, 9, 32])
def test_rows_by_the_statistics_of_their_blocks(rows, vocab):
    """Strips of weights leave each row's (maximum, sum) of 128 entries: whole and ragged blocks, more of them than threads hold, one entry
    more than a block.  Then choices that the short list of entries cannot hold: the same maximum once in every block, at
    another place in each (its lowest ids win, behind a few larger ones), all entries equal, and rows with fewer finite entries than candidates."""
    tune("ring_gemm", 0)
    if rows == 32 and vocab > 33000:
        vocab = 65537
    top_k = min(vocab, 16)
    x = _exact_inputs(rows, 128, vocab, vocab)
    _check(x, top_k=top_k, temperature=0.7, exact=True)
    _check(draft_head_inputs(rows, 128, vocab, seed=rows), top_k=top_k, temperature=1.3)
    x["f_top"][:] = 1.0
    one = np.zeros_like(x["w_head"][0])
    one[0] = 2.0
    x["w_head"][:] = 0.0
    for b in range(0, vocab, 128):
        x["w_head"][min(b + (37 * b // 128) % 128, vocab - 1)] = one
    _check(x, top_k=top_k, exact=True)
    for i, v in enumerate((vocab // 2, vocab - 1, vocab // 3)):
        x["w_head"][v] = one * (4.0 + i)
    _check(x, top_k=top_k, exact=True)
    x["w_head"][:] = 0.0
    lg, q, tk, tp = _check(x, top_k=top_k, exact=True)
    np.testing.assert_array_equal(tk, np.broadcast_to(np.arange(top_k), tk.shape))
    x["w_head"][:, 0] = -np.inf
    alive = sorted({vocab - 1, vocab // 2, 0})
    x["w_head"][alive] = one
    lg, q, tk, tp = _call(x, top_k=top_k)
    n = len(alive)
    assert (tk[:, :, :n] == np.array(alive)).all() and (tk[:, :, n:] == 0).all() and (tp[:, :, n:] == 0).all()
    np.testing.assert_allclose(tp[:, :, :n], 1.0 / n, rtol=1e-6)
    np.testing.assert_allclose(q[:, :, alive], 1.0 / n, rtol=1e-6)
    assert np.count_nonzero(q) == 2 * rows * n


@pytest.mark.parametrize("temperature", [4.3e-39, 4.2e-39, 3.5e-39, 2.95e-39])   # log2(e) / T beyond the largest float from 4.24e-39 downwards
def test_smallest_temperatures(temperature):
    """1 / T is a number down to 2.94e-39: rows of ordinary logits have the one distribution on their maximum, and rows whose logits are
    a few times 2^-126 apart (exact) an ordinary one."""
    tune("ring_gemm", 0)
    x = _exact_inputs(3, 128, 1001, 1)
    lg, q, tk, tp = _call(x, temperature=temperature)
    top = lg == lg.max(-1, keepdims=True)
    np.testing.assert_allclose(q, top / top.sum(-1, keepdims=True), rtol=1e-6)
    np.testing.assert_array_equal(tk, dh.top_candidates(lg, 5))
    np.testing.assert_allclose(tp, np.take_along_axis(q, tk.astype(np.int64), axis=-1), rtol=1e-6)
    x["f_top"][:] = 0.0
    x["f_top"][:, :, 0] = 1.0
    x["s_top"][:] = 1.0
    x["w_head"][:] = 0.0
    x["w_head"][:, 0] = np.arange(1001) % 9 * 2.0 ** -126
    lg, q, tk, tp = _call(x, temperature=temperature)
    np.testing.assert_array_equal(lg.astype(np.float64), np.broadcast_to(np.arange(1001) % 9 * 2.0 ** -126, lg.shape))
    # (against the reciprocal in 32 bits, which the division by a subnormal number does not have more of: a few roundings of exponents below 32)
    e = np.exp((lg.astype(np.float64) - 8 * 2.0 ** -126) * np.float64(np.float32(1.0) / np.float32(temperature)))
    np.testing.assert_allclose(q, e / e.sum(-1, keepdims=True), rtol=3e-5)
    np.testing.assert_allclose(tp, np.take_along_axis(q, tk.astype(np.int64), axis=-1), rtol=1e-6)


@pytest.mark.parametrize("rows,d,vocab,least", [(32, 128, 97144, 225280), (21, 512, 105552, 191744), (10, 4096, 128256, 335360), (3, 128, 1000, 2560)])
def test_the_least_workspace_serves_the_call(rows, d, vocab, least):
    """What the parts and their candidates take is enough, also where the statistics of the rows' blocks are more bytes; less is refused."""
    tune("ring_gemm", 0)
    g = torch.Generator(device="cuda").manual_seed(vocab)
    f = torch.randn((rows, 2, d), device="cuda", dtype=torch.bfloat16, generator=g)
    s = torch.rand((rows, 2), device="cuda", generator=g)
    w = torch.randn((vocab, d), device="cuda", dtype=torch.bfloat16, generator=g) * 5 * d ** -0.5

    def call(nbytes, guard=1024):
        room = torch.full((nbytes + guard,), 0xA5, dtype=torch.uint8, device="cuda")
        out = (torch.empty((rows, 2, vocab), device="cuda"), torch.empty((rows, 2, vocab), device="cuda"),
               torch.empty((rows, 2, 7), dtype=torch.int32, device="cuda"), torch.empty((rows, 2, 7), device="cuda"))
        jk.prepare_draft_heads(f, s, w, jk.JK_HEADS_DECOUPLED, 0.9, 7, 0.0, 0.0, *out, room[:nbytes]).launch()
        torch.cuda.synchronize()
        assert bool((room[nbytes:] == 0xA5).all())
        return out

    full = call(jk.draft_heads_workspace(rows, d, vocab))
    lg, q, tk, tp = call(least)
    assert torch.equal(lg, full[0]) and torch.equal(tk, full[2])
    torch.testing.assert_close(q, full[1], rtol=3e-5, atol=1e-30)
    torch.testing.assert_close(tp, full[3], rtol=3e-5, atol=1e-30)
    np.testing.assert_allclose(q.cpu().numpy(), dh.draft_distribution(lg.cpu().numpy(), 0.9), rtol=3e-5, atol=1e-30)
    with pytest.raises(jk.JakiroError):
        call(least - 256)


@pytest.mark.parametrize("vocab", [5, 300, 16385, 33000])
@pytest.mark.parametrize("rows", [1, 9, 32])
def test_statistics_of_rows_that_are_no_numbers(rows, vocab):
    """A NaN anywhere in a row, a block of nothing else and +inf make the whole distribution none, as the softmax of the same logits does; other
    rows stay what they are, and candidates are entries of the vocabulary."""
    tune("ring_gemm", 0)
    top_k = min(vocab, 8)

    def in_range(tk):
        assert ((tk >= 0) & (tk < vocab)).all()

    for first, n in ((vocab // 2, 1), (vocab // 128 // 2 * 128, 128)):   # an entry; a block
        x = _exact_inputs(rows, 128, vocab, vocab)
        x["w_head"][first:first + n] = np.nan
        lg, q, tk, tp = _call(x, top_k=top_k)
        assert np.isnan(lg[:, :, first:first + n]).all() and np.isnan(q).all()
        in_range(tk)
    x = _exact_inputs(rows, 128, vocab, vocab)
    x["f_top"][:, :, 7] = 0.0
    good = _call(x, top_k=top_k)
    for column, low in ((1.0, -1.0), (0.0, -1.0), (0.0, 0.5)):   # +inf and -inf; NaN and -inf; NaN and +inf
        x["w_head"][:, 7] = low
        x["w_head"][vocab // 3, 7] = column
        x["f_top"][0, 0, 7] = np.inf
        lg, q, tk, tp = _call(x, top_k=top_k)
        assert not np.isfinite(lg[0, 0]).any() and np.isnan(q[0, 0]).all()
        in_range(tk)
        for got, ref in zip((lg, q, tk, tp), good):
            np.testing.assert_array_equal(got[0, 1], ref[0, 1])
            np.testing.assert_array_equal(got[1:], ref[1:])
