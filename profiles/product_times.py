"""Times of the draft side's products by either of the two kernels that can compute them, and what the library's choice between
them is worth.

    python profiles/product_times.py measure OUT.csv [SHAPES] [SEED]    on an MI355X (about a minute per 1000 shapes)
    python profiles/product_times.py report [CSV]                       anywhere; default: product_times.csv

A shape is a whole call of `jk_draft_heads` (1 - 16 tokens), `jk_moe_experts` (1 - 80 rows) or `jk_linear` (1 - 128 rows); `strips` is
its time with every product on stream_gemm.hip, `other` with every product on ring_gemm.hip (heads, experts) or on the kernel of few
columns (linear layers; 0: cannot be), `auto` as the library chooses, for the experts' two launches apart.  (`jk_set_tuning`: ring_gemm,
narrow_gemm.)  A time is the median of five HIP-graph replays over a ring of up to sixteen different weights (500 MB together where
they are large), so that large weights come from HBM and small ones from the Infinity Cache.
"""
import csv
import math
import os
import random
import statistics
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
FIELDS = ("kind", "rows", "k", "n", "experts", "strips", "other", "auto")


def shapes(count, seed):
    rng = random.Random(seed)

    def spread(lo, hi):
        return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))

    while count > 0:
        kind = rng.choice(["heads", "experts", "experts", "linear"])
        experts = 0
        if kind == "heads":
            rows, k, n = spread(1, 16), 128 * spread(4, 64), spread(8192, 128256)
        elif kind == "experts":
            rows, k, n, experts = spread(1, 80), 128 * spread(4, 64), 128 * spread(4, 112), rng.choice([2, 4, 5, 8, 8])
        else:
            rows, k, n = spread(1, 128), 128 * spread(4, 128), 4 * spread(128, 4096)
        if k * n * max(1, 3 * experts) <= 4e8:
            count -= 1
            yield kind, rows, k, n, experts


def measure(path, count, seed):
    sys.path.insert(0, os.path.dirname(HERE))
    import torch

    import paper_2502_06282_amd as jk

    def elapsed(graph, reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(reps):
            graph.replay()
        b.record()
        torch.cuda.synchronize()
        return a.elapsed_time(b) * 1e3 / reps

    pool = torch.randn(900_000_000, device="cuda", dtype=torch.bfloat16)
    pool *= 0.02
    with open(path, "w", newline="") as f:
        out = csv.writer(f)
        out.writerow(FIELDS)
        for i, (kind, rows, k, n, experts) in enumerate(shapes(count, seed)):
            size = k * n * max(1, 3 * experts)
            ring = max(1, min(16, int(250e6 / size)))
            weights = [pool[j * size:(j + 1) * size] for j in range(ring)]
            x = torch.randn((rows, 2, k), device="cuda").to(torch.bfloat16)
            score = torch.rand((rows, 2), device="cuda")
            centroids = torch.randn((max(experts, 1), k), device="cuda").mul_(0.02).to(torch.bfloat16)

            def call(w):
                if kind == "heads":
                    jk.draft_heads(x, score, w.view(n, k), jk.JK_HEADS_DECOUPLED, 1.0, 8)
                elif kind == "experts":
                    gate, up, down = w.view(3, experts, -1)
                    jk.moe_experts(x[:, 0].contiguous(), centroids, gate.view(experts, n, k), up.view(experts, n, k), down.view(experts, k, n))
                else:
                    jk.linear(x[:, 0].contiguous(), w.view(n, k))

            us = []
            for forced in (0, 1, -1):
                jk.set_tuning("ring_gemm", forced)
                jk.set_tuning("narrow_gemm", forced)
                if forced == 1 and kind == "linear" and n > 64 * 256:
                    us.append(0.0)
                    continue
                call(weights[0])
                torch.cuda.synchronize()
                graph = torch.cuda.CUDAGraph()
                with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
                    for w in weights:
                        call(w)
                graph.replay()
                reps = max(1, min(30, int(2000 / max(1.0, elapsed(graph, 1)))))
                us.append(statistics.median(elapsed(graph, reps) for _ in range(5)) / ring)
            out.writerow((kind, rows, k, n, experts, *(f"{t:.2f}" for t in us)))
            f.flush()
            if i % 100 == 99:
                print(i + 1, "shapes", flush=True)
    for name in ("ring_gemm", "narrow_gemm"):
        jk.set_tuning(name, -1)


def report(path):
    with open(path) as f:
        rows = [r for r in csv.DictReader(f) if float(r["other"]) > 0]
    for kind in ("heads", "experts", "linear"):
        t = [tuple(float(r[x]) for x in FIELDS[5:]) for r in rows if r["kind"] == kind]
        gain = sorted(s / a for s, _, a in t)
        loss = sorted(a / min(s, o, a) for s, o, a in t)
        geo = lambda v: math.exp(statistics.fmean(map(math.log, v)))
        at = lambda v, q: v[min(len(v) - 1, int(q * len(v)))]
        print(f"{kind}: {len(t)} shapes.  The choice against strips alone: {geo(gain):.3f} times as fast, 1st percentile {at(gain, 0.01):.3f}, "
              f"5th {at(gain, 0.05):.3f}, least {gain[0]:.3f}; against the other kernel alone {geo([o / a for _, o, a in t]):.3f}; behind the "
              f"best of the three: geometric mean {geo(loss):.4f}, 95th percentile {at(loss, 0.95):.3f}, worst {loss[-1]:.3f}")


if __name__ == "__main__":
    if len(sys.argv) >= 3 and sys.argv[1] == "measure":
        measure(sys.argv[2], int(sys.argv[3]) if len(sys.argv) > 3 else 1000, int(sys.argv[4]) if len(sys.argv) > 4 else 1)
    elif len(sys.argv) >= 2 and sys.argv[1] == "report":
        report(sys.argv[2] if len(sys.argv) > 2 else os.path.join(HERE, "product_times.csv"))
    else:
        sys.exit(__doc__)
