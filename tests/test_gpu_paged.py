"""GPU parity for the paged KV cache: jk_tree_verify_attention_paged against the attention oracle on
the cache read back in table order, bitwise against the contiguous call on the same data, and
jk_commit_path_layers_paged against the commit oracle at the paged addresses."""
import numpy as np
import pytest
import torch

import paper_2502_06282_amd as jk
from gpu_util import reset_tuning, tune
from oracle import commit_path as oracle_commit, gather_pages, tree_verify_attention as oracle_attention
from workloads import CONFIGS, attention_inputs, paged_layout, round_to_bf16, tree_for_config

pytestmark = pytest.mark.gpu
BF = torch.bfloat16


def _dev(a, dtype=BF):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda().to(dtype)


def _paged_case(cfg, page_size, L, seed=0):
    par = tree_for_config(cfg, seed=seed)
    x = {k: round_to_bf16(v) for k, v in attention_inputs(cfg, seed=seed, prefix_len=L, scale_mult=np.sqrt(128.0)).items()}
    (kp, vp), table = paged_layout(x["k_cache"], x["v_cache"], page_size, seed=seed)
    return par, x, kp, vp, table


@pytest.mark.parametrize("wm,wn", [(2, 2), (4, 1)], ids=["2x2", "4x1"])
@pytest.mark.parametrize("page_size,L", [(32, 97), (64, 300), (128, 1000), (32, 0), (256, 515)])
def test_paged_attention_matches_oracle_and_contiguous(monkeypatch, wm, wn, page_size, L):
    tune("attn_wm", str(wm))
    tune("attn_wn", str(wn))
    cfg = CONFIGS["c3_llama3_8b"].with_(batch=2, prefix_len=L, n_q_heads=8, n_kv_heads=2)
    par, x, kp, vp, table = _paged_case(cfg, page_size, max(L, 1), seed=L + page_size)
    plen = [L, L // 3]
    ref = oracle_attention(**x, parent=par, prefix_len=plen)
    parent = torch.from_numpy(par).cuda()
    pl = torch.tensor(plen, dtype=torch.int32).cuda()
    for s in ("1", "3"):
        tune("attn_splits", s)
        got = jk.tree_verify_attention_paged(_dev(x["q"]), _dev(kp), _dev(vp), torch.from_numpy(table).cuda(),
                                             _dev(x["k_tree"]), _dev(x["v_tree"]), parent, pl, max_prefix_len=max(L, 1))
        cont = jk.tree_verify_attention(_dev(x["q"]), _dev(x["k_cache"]), _dev(x["v_cache"]), _dev(x["k_tree"]),
                                        _dev(x["v_tree"]), parent, pl, max_prefix_len=max(L, 1))
        torch.cuda.synchronize()
        g = got.float().cpu().numpy()
        assert np.isfinite(g).all()            # the NaN-filled spare pages and page tails were never read
        assert np.abs(g - ref).max() <= 2e-2
        assert torch.equal(got, cont)          # same arithmetic in the same order, only the addresses differ


@pytest.mark.parametrize("wm,wn", [(2, 2), (4, 1), (8, 1)], ids=["2x2", "4x1", "8x1"])
@pytest.mark.parametrize("plen", [(9001, 8300), (9001, 9001), (33, 9001)], ids=["ragged", "equal", "swapped"])
@pytest.mark.parametrize("Hkv", [8, 2])
def test_paged_batch_with_more_pages_than_threads(Hkv, wm, wn, plen):
    """Page ids come a thread's first one at once, and what lies past 256 of them in turn.  A batch whose KV heads are a multiple of
    eight together asks for them when its lengths are there; another one (arrangements of up to 128 rows), as if all had the bound's
    length, and those below it make their list again, here of more than 256 too.  Bitwise equal to the contiguous call."""
    tune("attn_wm", str(wm))
    tune("attn_wn", str(wn))
    tune("attn_splits", "1")
    g = torch.Generator(device="cuda").manual_seed(sum(plen))
    B, T, H, D, L, page = 2, 40, 4 * Hkv, 128, max(plen), 32
    par = torch.from_numpy(np.stack([tree_for_config(CONFIGS["c3_llama3_8b"].with_(n_tree=T), seed=b)[0] for b in range(B)])).cuda()
    blocks = -(-L // page)
    rand = lambda *s: torch.randn(s, device="cuda", generator=g).to(BF)
    kp, vp = rand(B * blocks + 5, page, Hkv, D), rand(B * blocks + 5, page, Hkv, D)
    table = torch.randperm(B * blocks + 5, device="cuda", generator=g)[:B * blocks].reshape(B, blocks).to(torch.int32).contiguous()
    kc, vc = (x[table.long()].reshape(B, blocks * page, Hkv, D)[:, :L].contiguous() for x in (kp, vp))
    q, kt, vt = rand(B, T, H, D), rand(B, T, Hkv, D), rand(B, T, Hkv, D)
    pl = torch.tensor(plen, dtype=torch.int32, device="cuda")
    got = jk.tree_verify_attention_paged(q, kp, vp, table, kt, vt, par, pl, max_prefix_len=L)
    cont = jk.tree_verify_attention(q, kc, vc, kt, vt, par, pl, max_prefix_len=L)
    torch.cuda.synchronize()
    assert torch.isfinite(got.float()).all() and torch.equal(got, cont)


def test_paged_attention_repeats_a_split_that_leaves_the_fixed_frame(monkeypatch):
    """A late key far above everything before it for one query row: the two-tile fast path of the 4x1
    arrangement gives up and the workgroup streams its split again on the general path, through the page
    table once more.  Bitwise equal to the contiguous call, which takes the same decisions."""
    tune("attn_wm", "4")
    tune("attn_wn", "1")
    tune("attn_splits", "2")
    cfg = CONFIGS["c3_llama3_8b"].with_(batch=1, prefix_len=2048, n_q_heads=8, n_kv_heads=2)
    par = tree_for_config(cfg, seed=3)
    x = {k: round_to_bf16(v) for k, v in attention_inputs(cfg, seed=3, scale_mult=np.sqrt(128.0)).items()}
    x["k_cache"][0, 1777, 0] = round_to_bf16(8.0 * x["q"][0, 11, 2])
    (kp, vp), table = paged_layout(x["k_cache"], x["v_cache"], 64, seed=3)
    ref = oracle_attention(**x, parent=par, prefix_len=[2048])
    parent = torch.from_numpy(par).cuda()
    pl = torch.tensor([2048], dtype=torch.int32).cuda()
    got = jk.tree_verify_attention_paged(_dev(x["q"]), _dev(kp), _dev(vp), torch.from_numpy(table).cuda(),
                                         _dev(x["k_tree"]), _dev(x["v_tree"]), parent, pl, max_prefix_len=2048)
    cont = jk.tree_verify_attention(_dev(x["q"]), _dev(x["k_cache"]), _dev(x["v_cache"]), _dev(x["k_tree"]),
                                    _dev(x["v_tree"]), parent, pl, max_prefix_len=2048)
    torch.cuda.synchronize()
    g = got.float().cpu().numpy()
    assert np.isfinite(g).all()
    assert np.abs(g - ref).max() <= 3 * 2.0 ** -8 * 4.5 and np.abs(g - ref).max() <= 1.5e-2 * np.abs(ref).max()
    v = x["v_cache"][0, 1777, 0].astype(np.float64)
    assert np.abs(g[0, 11, 2] - v).max() <= 2.0 ** -7 * np.abs(v).max() + 1e-6
    assert torch.equal(got, cont)


def test_paged_attention_full_size_c3():
    cfg = CONFIGS["c3_llama3_8b"]
    par, x, kp, vp, table = _paged_case(cfg, 128, cfg.prefix_len)
    parent = torch.from_numpy(par).cuda()
    pl = torch.tensor([cfg.prefix_len], dtype=torch.int32).cuda()
    got = jk.tree_verify_attention_paged(_dev(x["q"]), _dev(kp), _dev(vp), torch.from_numpy(table).cuda(),
                                         _dev(x["k_tree"]), _dev(x["v_tree"]), parent, pl, max_prefix_len=cfg.prefix_len)
    cont = jk.tree_verify_attention(_dev(x["q"]), _dev(x["k_cache"]), _dev(x["v_cache"]), _dev(x["k_tree"]),
                                    _dev(x["v_tree"]), parent, pl)
    torch.cuda.synchronize()
    assert torch.equal(got, cont)
    kv = 5
    G = cfg.group
    sub = {"q": x["q"][:, :, kv * G:(kv + 1) * G], "k_cache": x["k_cache"][:, :, kv:kv + 1], "v_cache": x["v_cache"][:, :, kv:kv + 1],
           "k_tree": x["k_tree"][:, :, kv:kv + 1], "v_tree": x["v_tree"][:, :, kv:kv + 1]}
    ref = oracle_attention(**sub, parent=par, prefix_len=[cfg.prefix_len])
    assert np.abs(got.float().cpu().numpy()[0, :, kv * G:(kv + 1) * G] - ref[0]).max() <= 2e-2


def test_paged_commit_all_layers():
    cfg = CONFIGS["c2_vicuna7b"].with_(batch=2, prefix_len=160, n_q_heads=4, n_kv_heads=4)
    page = 32
    rng = np.random.default_rng(9)
    n_layers = 3
    xs = [{k: round_to_bf16(v) for k, v in attention_inputs(cfg, layer=l).items()} for l in range(n_layers)]
    layouts = [paged_layout(x["k_cache"], x["v_cache"], page, seed=1) for x in xs]   # same table for all layers
    table = layouts[0][1]
    path = np.full((2, cfg.depth), -1, dtype=np.int32)
    path[0, :4] = [3, 9, 20, 41]
    path[1, :2] = [0, 7]
    alen, plen = [4, 2], [94, 158]          # sequence 0 crosses a page boundary (96); sequence 1 ends the cache
    kps = [_dev(l[0][0]) for l in layouts]
    vps = [_dev(l[0][1]) for l in layouts]
    kts, vts = [_dev(x["k_tree"]) for x in xs], [_dev(x["v_tree"]) for x in xs]
    p = torch.from_numpy(path).cuda()
    al = torch.tensor(alen, dtype=torch.int32).cuda()
    pl = torch.tensor(plen, dtype=torch.int32).cuda()
    jk.prepare_commit_path_layers_paged(kts, vts, kps, vps, torch.from_numpy(table).cuda(), p, al, pl).launch()
    torch.cuda.synchronize()
    for l, x in enumerate(xs):
        rk, rv, rl = oracle_commit(x["k_cache"], x["v_cache"], x["k_tree"], x["v_tree"], path, alen, plen)
        gk = gather_pages(kps[l].float().cpu().numpy(), table, page, 160)
        gv = gather_pages(vps[l].float().cpu().numpy(), table, page, 160)
        np.testing.assert_array_equal(gk, rk.astype(np.float32))
        np.testing.assert_array_equal(gv, rv.astype(np.float32))
        # spare pages stay NaN: nothing was written outside the sequences' own pages
        used = set(table.ravel().tolist())
        spare = [i for i in range(kps[l].shape[0]) if i not in used]
        assert torch.isnan(kps[l][spare].float()).all()
    np.testing.assert_array_equal(pl.cpu().numpy(), rl)


def test_paged_argument_errors():
    cfg = CONFIGS["c2_vicuna7b"].with_(batch=1, prefix_len=64, n_q_heads=4, n_kv_heads=4)
    par, x, kp, vp, table = _paged_case(cfg, 48, 64)      # 48 is not a multiple of 32
    parent = torch.from_numpy(par).cuda()
    pl = torch.tensor([64], dtype=torch.int32).cuda()
    with pytest.raises(jk.JakiroError):
        jk.tree_verify_attention_paged(_dev(x["q"]), _dev(kp), _dev(vp), torch.from_numpy(table).cuda(), _dev(x["k_tree"]),
                                       _dev(x["v_tree"]), parent, pl, max_prefix_len=64)
    par, x, kp, vp, table = _paged_case(cfg, 32, 64)
    with pytest.raises(jk.JakiroError):                    # the table cannot hold max_prefix_len tokens
        jk.tree_verify_attention_paged(_dev(x["q"]), _dev(kp), _dev(vp), torch.from_numpy(table).cuda(), _dev(x["k_tree"]),
                                       _dev(x["v_tree"]), parent, pl, max_prefix_len=200)


def test_paged_table_entries_past_a_sequences_pages_may_hold_anything():
    """The first transfers go out on the assumption prefix_len == max_prefix_len, through whatever the table
    holds for those pages (ids are clamped into the pool).  With one sequence much shorter than the bound and
    wild values behind its pages, the results are those of a clean table, bit for bit, and the error word
    stays clear: nothing past a sequence's pages reaches a result."""
    cfg = CONFIGS["c3_llama3_8b"].with_(batch=2, prefix_len=1500, n_q_heads=8, n_kv_heads=2)
    page = 64
    par, x, kp, vp, table = _paged_case(cfg, page, 1500, seed=7)
    plen = [1500, 200]
    dirty = table.copy()
    used = (200 + page - 1) // page
    dirty[1, used:] = np.array([-5, 2 ** 30, -2 ** 31, 123456789] * 8, dtype=np.int32)[: dirty.shape[1] - used]
    parent = torch.from_numpy(par).cuda()
    pl = torch.tensor(plen, dtype=torch.int32).cuda()
    ref = oracle_attention(**x, parent=par, prefix_len=plen)
    for arr in ((4, 1), (2, 2)):
        for s in (1, 3):
            tune("attn_wm", arr[0]); tune("attn_wn", arr[1]); tune("attn_splits", s)
            outs = []
            for tab in (table, dirty):
                q = _dev(x["q"])
                need = jk.tree_verify_attention_workspace(q, _dev(x["k_cache"]), _dev(x["k_tree"]), 1500)
                ws = torch.zeros(need, dtype=torch.uint8, device="cuda")
                outs.append(jk.tree_verify_attention_paged(q, _dev(kp), _dev(vp), torch.from_numpy(tab).cuda(), _dev(x["k_tree"]),
                                                           _dev(x["v_tree"]), parent, pl, max_prefix_len=1500, workspace=ws))
                torch.cuda.synchronize()
                assert jk.last_device_error(ws) == 0
            assert torch.equal(outs[0], outs[1])
            assert np.abs(outs[1].float().cpu().numpy() - ref).max() <= 2e-2


def test_paged_page_id_outside_the_pool_is_clamped_and_reported():
    """An id outside [0, n_pages) among a sequence's own pages: the transfer stays inside the pool (the id is clamped
    to its nearest end), the result is that of the clamped table, and JK_DEVERR_BAD_PAGE is set; a clean table leaves
    the word clear."""
    cfg = CONFIGS["c3_llama3_8b"].with_(batch=2, prefix_len=700, n_q_heads=8, n_kv_heads=2)
    page = 64
    par, x, kp, vp, table = _paged_case(cfg, page, 700, seed=13)
    kp, vp = np.nan_to_num(kp, nan=0.0), np.nan_to_num(vp, nan=0.0)      # (a clamped id lands on some real page: keep it finite)
    n_pages = kp.shape[0]
    bad = table.copy()
    bad[0, 3] = n_pages + 50
    bad[1, 0] = -9
    fixed = bad.copy()
    fixed[0, 3] = n_pages - 1
    fixed[1, 0] = 0
    parent = torch.from_numpy(par).cuda()
    pl = torch.tensor([700, 650], dtype=torch.int32).cuda()
    for arr, s in (((4, 1), 1), ((4, 1), 3), ((2, 2), 2)):
        tune("attn_wm", arr[0]); tune("attn_wn", arr[1]); tune("attn_splits", s)
        outs, errs = [], []
        for tab in (bad, fixed, table):
            q = _dev(x["q"])
            ws = torch.zeros(jk.tree_verify_attention_workspace(q, _dev(x["k_cache"]), _dev(x["k_tree"]), 700), dtype=torch.uint8,
                             device="cuda")
            outs.append(jk.tree_verify_attention_paged(q, _dev(kp), _dev(vp), torch.from_numpy(tab).cuda(), _dev(x["k_tree"]),
                                                       _dev(x["v_tree"]), parent, pl, max_prefix_len=700, workspace=ws))
            torch.cuda.synchronize()
            errs.append(jk.last_device_error(ws))
        assert errs == [jk.JK_DEVERR_BAD_PAGE, 0, 0], (arr, s, errs)
        assert torch.equal(outs[0], outs[1])
        assert not torch.equal(outs[0], outs[2])


@pytest.mark.parametrize("hkv,lens", [
    (8, [700, 0, 33, 512, 1, 640, 31, 257]),
    (4, [0, 900]),
    (8, [65, 64]),
    (16, [300, 300, 300]),
    (2, [600, 10, 10, 600, 599, 601, 0, 32, 33, 96, 128, 1]),
    (1, [(37 * i) % 400 for i in range(64)]),
    (1, [(53 * i) % 300 for i in range(72)]),
], ids=["eight", "two", "one-key-apart", "equal", "ties", "sixty-four", "more-than-lanes"])
def test_sequences_of_a_batch_give_what_each_gives_alone(hkv, lens):
    """The workgroups of a batch take its sequences by falling length (up to 64 of them, where the KV heads of the
    batch divide by eight).  Whatever the order: bit for bit the result of the sequence in a call of its own, paged
    or not, with the splits merged in the kernel and by the second one, in a workspace used again with other
    lengths."""
    B, L, G, T = len(lens), max(lens), 2, 20
    cfg = CONFIGS["c3_llama3_8b"].with_(batch=B, prefix_len=L, n_q_heads=hkv * G, n_kv_heads=hkv, n_tree=T)
    par, x, kp, vp, table = _paged_case(cfg, 32, L, seed=B)
    d = {k: _dev(v) for k, v in x.items()}
    kp, vp, table, parent = _dev(kp), _dev(vp), torch.from_numpy(table).cuda(), torch.from_numpy(par).cuda()
    ref = oracle_attention(**x, parent=par, prefix_len=lens)
    bound = L + 5  # (no sequence is as long as the bound)
    for wm, splits, fused in ((2, 1, -1), (4, 1, -1), (2, 3, 0), (4, 3, 1)):
        tune("attn_wm", wm); tune("attn_wn", 4 // wm); tune("attn_splits", splits); tune("attn_fused", fused)
        ws = torch.empty(jk.tree_verify_attention_workspace(d["q"], d["k_cache"], d["k_tree"], bound), dtype=torch.uint8, device="cuda")
        jk.workspace_init(ws)
        for most, order in ((L, list(range(B))), (L, list(range(B))[::-1]), (bound, list(range(B)))):
            pl = torch.tensor([lens[i] for i in order], dtype=torch.int32).cuda()
            pick = torch.tensor(order).cuda()
            a = [d[k][pick].contiguous() for k in ("q", "k_cache", "v_cache", "k_tree", "v_tree")]
            if most > L:
                a[1], a[2] = (torch.nn.functional.pad(t, (0, 0, 0, 0, 0, most - L)) for t in (a[1], a[2]))
            got = jk.tree_verify_attention(*a, parent[pick].contiguous(), pl, max_prefix_len=most, workspace=ws)
            if most == L:
                paged = jk.tree_verify_attention_paged(a[0], kp, vp, table[pick].contiguous(), a[3], a[4], parent[pick].contiguous(), pl,
                                                       max_prefix_len=most, workspace=ws)
                assert torch.equal(got, paged)
            g = got.float().cpu().numpy()
            assert np.isfinite(g).all() and np.abs(g - ref[order]).max() <= 2e-2
            tune("attn_fused", 0)
            for i in (0, B // 2, B - 1):
                alone = jk.tree_verify_attention(*(t[i:i + 1].contiguous() for t in a), parent[pick][i:i + 1].contiguous(), pl[i:i + 1],
                                                 max_prefix_len=most)
                same = torch.equal(got[i:i + 1], alone) if fused != 1 else (got[i:i + 1].float() - alone.float()).abs().max() <= 2e-2
                assert same, (wm, splits, fused, most, i)
            tune("attn_fused", fused)
        assert jk.last_device_error(ws) == 0
