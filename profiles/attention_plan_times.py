"""Times of many launch plans of drawn attention shapes, and how far the library's own choice is from the best of them.

    python profiles/attention_plan_times.py measure OUT.csv [SHAPES] [SEED]    on an MI355X (about a minute per 1000 shapes)
    python profiles/attention_plan_times.py report [CSV]                       anywhere; default: attention_plan_times.csv

A shape is a bf16 call of `jk_tree_verify_attention` (batch 1 - 32, 1 - 128 tree nodes, the head counts of the workloads,
head_dim 64 or 128, prefixes of 64 - 32768 tokens, all sequences of a batch equally long); a plan is a wave arrangement
and a number of key splits (`jk_set_tuning`), up to 22 of them per shape, always with one split, two, and the choice of
the plan itself.  A time is the median of three HIP-graph replays over a ring of up to sixteen different K/V caches
(600 MB together where they are large), so that large caches come from HBM and small ones from the Infinity Cache.
"""
import csv
import math
import os
import random
import statistics
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
FIELDS = ("batch", "n_tree", "hq", "hkv", "d", "prefix", "wm", "wn", "splits", "fused", "chosen", "us")
SPLITS = (1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 16, 18, 21, 24, 28, 32, 40, 48, 64)


def shapes(n, seed):
    rng = random.Random(seed)

    def spread(lo, hi):
        return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))

    while n > 0:
        hq, hkv = rng.choice([(32, 32), (32, 8), (40, 40), (64, 8), (16, 2), (8, 8)])
        s = (spread(1, 32), spread(1, 8) if rng.random() < 0.25 else spread(8, 128), hq, hkv, rng.choice([64, 128, 128]), spread(64, 32768))
        b, t, _, _, d, length = s
        if 4 * b * length * hkv * d <= 1.2e9 and 4 * b * t * hq * d * length <= 4e12:
            n -= 1
            yield s


def candidates(shape, chosen, rng):
    b, t, hq, hkv, _, length = shape
    rows, top = t * hq // hkv, max(1, min(64, (-(-length // 32) - (-t // 32)) // 4))
    out = []
    tiles = -(-length // 32) - (-t // 32)
    for wm, wn in ((2, 2), (4, 1), (8, 1)):
        if wm == 8 and rows <= 96 or wm == 4 and rows <= 64:
            continue
        wgs = b * hkv * -(-rows // (32 * wm))
        fit = {max(1, round(x * 256 / wgs)) for x in (0.5, 1, 1.5, 2, 3, 4)}  # a workgroup for that many times the CUs
        out += [(wm, wn, s) for s in sorted(fit.union(SPLITS)) if s <= top and wgs * s <= 3072 and (s == 1 or wgs * s >= 64 or s >= top // 2)]
    if tiles <= 56:  # (undivided; the plan takes it up to 28)
        out.append((1, 4, 1))
    keep = sorted({chosen, *(c for c in out if c[2] <= 2)})
    rest = [c for c in out if c not in keep]
    rng.shuffle(rest)
    return sorted(keep + rest[:22 - len(keep)])


def measure(path, n, seed):
    sys.path.insert(0, os.path.dirname(HERE))
    import torch

    import paper_2502_06282_amd as jk

    def force(wm, wn, splits):
        for name, v in (("attn_wm", wm), ("attn_wn", wn), ("attn_splits", splits)):
            jk.set_tuning(name, v)

    def elapsed(graph, reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(reps):
            graph.replay()
        b.record()
        torch.cuda.synchronize()
        return a.elapsed_time(b) * 1e3 / reps

    pool = torch.randn(900_000_000, device="cuda", dtype=torch.bfloat16)
    rng = random.Random(seed + 1)
    with open(path, "w", newline="") as f:
        out = csv.writer(f)
        out.writerow(FIELDS)
        for k, shape in enumerate(shapes(n, seed)):
            b, t, hq, hkv, d, length = shape
            size = b * length * hkv * d
            ring = max(1, min(16, int(150e6 / size)))
            caches = [[pool[(2 * i + j) * size:(2 * i + j + 1) * size].view(b, length, hkv, d) for j in (0, 1)] for i in range(ring)]
            q, kt = pool[-b * t * hq * d:].view(b, t, hq, d), pool[-b * t * hkv * d:].view(b, t, hkv, d)
            o = torch.empty_like(q)
            parent = torch.tensor([[max(-1, i // 2 - 1) for i in range(t)]] * b, dtype=torch.int32, device="cuda")
            plen = torch.full((b,), length, dtype=torch.int32, device="cuda")
            force(0, 0, 0)
            p = jk.tree_verify_attention_plan(q, caches[0][0], kt, length)
            chosen = (p["wm"], p["wn"], p["splits"])
            for plan in candidates(shape, chosen, rng):
                force(*plan)
                try:
                    p = jk.tree_verify_attention_plan(q, caches[0][0], kt, length)
                except jk.JakiroError:
                    continue  # (more partial results than that kernel merges)
                if (p["wm"], p["wn"], p["splits"]) != plan:
                    continue  # (a split has a least number of tiles)
                ws = torch.empty(jk.tree_verify_attention_workspace(q, caches[0][0], kt, length), dtype=torch.uint8, device="cuda")
                jk.workspace_init(ws)

                def call(c):
                    jk.tree_verify_attention(q, c[0], c[1], kt, kt, parent, plen, max_prefix_len=length, out=o, workspace=ws)

                call(caches[0])
                torch.cuda.synchronize()
                graph = torch.cuda.CUDAGraph()
                with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
                    for c in caches:
                        call(c)
                graph.replay()
                reps = max(1, min(20, int(1500 / max(1.0, elapsed(graph, 1)))))
                us = statistics.median(elapsed(graph, reps) for _ in range(3)) / ring
                out.writerow((*shape, *plan, p["fused"], int(plan == chosen), f"{us:.2f}"))
            f.flush()
            if k % 100 == 99:
                print(k + 1, "shapes", flush=True)
    force(0, 0, 0)


def report(path):
    plans = {}
    with open(path) as f:
        for r in csv.DictReader(f):
            plans.setdefault(tuple(int(r[x]) for x in FIELDS[:6]), []).append((int(r["chosen"]), float(r["us"])))
    loss = sorted(next(us for c, us in p if c) / min(us for _, us in p) for p in plans.values())
    mean = math.exp(statistics.fmean(map(math.log, loss)))
    at = lambda q: loss[min(len(loss) - 1, int(q * len(loss)))]
    print(f"{len(loss)} shapes, {sum(map(len, plans.values()))} plans; the chosen plan against the best one timed: geometric mean "
          f"{mean:.4f}, median {at(0.5):.3f}, 90th percentile {at(0.9):.3f}, 99th {at(0.99):.3f}, worst {loss[-1]:.3f}")


if __name__ == "__main__":
    if len(sys.argv) >= 3 and sys.argv[1] == "measure":
        measure(sys.argv[2], int(sys.argv[3]) if len(sys.argv) > 3 else 1000, int(sys.argv[4]) if len(sys.argv) > 4 else 1)
    elif len(sys.argv) >= 2 and sys.argv[1] == "report":
        report(sys.argv[2] if len(sys.argv) > 2 else os.path.join(HERE, "attention_plan_times.csv"))
    else:
        sys.exit(__doc__)
