"""Offline tile sweep: time every GEMM tile on each workload shape and write the
per-shape table (tile_table.inc) the library compiles in.

The paper tunes its kernel per (M, N, K) with an autotuner over 36 configurations at
first call (Section 3, "Why autotuning is load-bearing"); here the search runs once,
offline, on the target GPU, and its result is a constant table in the library.

Two sets of shapes: the workload shapes (one entry each, for their exact M) and the
paper's five model shapes over its token counts (Section 3, "Target architecture";
Section 5), which get token-count buckets: each swept M owns the range up to the
midpoints with its neighbours.

The cost models that choose a plan for the other shapes (kTileCost, kStreamCost) are
fitted to random shapes: --random N times every modeled tile and the default plan on N of
them, --fit fits both models to saved sweeps and says how far the default plan and the
fallback tile are from the fastest one measured.

Usage (on an MI355X): python -m paper_2606_14598_amd.tune --out tile_table.inc
       [--json r.json] [--set all|workloads|paper] [--iters N]
       python -m paper_2606_14598_amd.tune --random N [--seed S] [--m-max M] --json r.json
       python -m paper_2606_14598_amd.tune --fit r.json [r2.json ...]        (no GPU)
"""
from __future__ import annotations

import argparse
import json
import math
import os
import random
import re
import sys

import numpy as np
import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

import paper_2606_14598_amd as w8a8  # noqa: E402
import synth_inputs as si  # noqa: E402

HEADER = """// Offline-chosen GEMM tile per shape: {M lower bound, M upper bound, N, K, tile id}.
// Written by paper_2606_14598_amd/tune.py from a timed sweep of every tile on MI355X;
// shapes not listed, and those above 16 tokens where a plan is predicted clearly faster, use
// the cost models below (gemm_i8.hip).
"""

CUS = 256


def time_ms(fn, iters=20, warmup=3, warm_ms=0.0, min_timed_ms=2.0):
    """Mean ms per call of fn: `iters` calls captured once in a HIP graph and replayed,
    so microsecond kernels are timed without the host's per-launch overhead. The graph
    is replayed for `warm_ms` before timing, and timed over at least `min_timed_ms`."""
    for _ in range(warmup):
        fn()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            for _ in range(iters):
                fn()
    st, en = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    st.record()
    g.replay()
    en.record()
    torch.cuda.synchronize()
    once = max(st.elapsed_time(en), 1e-3)
    for _ in range(int(warm_ms / once)):
        g.replay()
    reps = max(3, int(min_timed_ms / once) + 1)
    torch.cuda.synchronize()
    st.record()
    for _ in range(reps):
        g.replay()
    en.record()
    torch.cuda.synchronize()
    return st.elapsed_time(en) / (reps * iters)


def shapes(which: str = "all"):
    """(shape, M lower bound, M upper bound) of every entry to tune."""
    seen = set()
    if which in ("all", "workloads"):
        for c in sorted(si.WORKLOADS):
            for s in si.WORKLOADS[c]:
                key = (s.M, s.N, s.K)
                if key not in seen:
                    seen.add(key)
                    yield s, s.M, s.M
    if which in ("all", "paper"):
        ms = sorted(si.PAPER_M)
        for name, _, _ in si.PAPER_SHAPES:
            for i, M in enumerate(ms):
                lo = 257 if i == 0 else (ms[i - 1] + M) // 2 + 1
                hi = (1 << 62) if i == len(ms) - 1 else (M + ms[i + 1]) // 2
                yield si.paper_shape(name, M), lo, hi


def _dev_bf16(bits, dev):
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).view(torch.bfloat16).to(dev)


def sweep(iters: int, which: str = "all"):
    """Time every tile on every shape, on the shape's own synthetic inputs quantized by
    the library: the matrix cores' sustained rate depends on the operand bits
    (switching power), so uniform random or constant codes would mislead. The
    weight-streaming tiles (made for M <= 128) are skipped above 128 tokens, and the
    split-K tiles where their unsplit tile already gives two workgroups per CU. The chip's
    power management needs ~15-20 ms of sustained load to settle after an idle gap (the
    input generation between shapes is one), so each shape first runs 30 ms of work,
    and every tile is timed twice, in two passes, keeping the faster."""
    dev = torch.device("cuda:0")
    results = []
    for s, lo, hi in shapes(which):
        x, w, bb = si.make_inputs(s)
        xd = _dev_bf16(x, dev)
        del x
        xq, sx = w8a8.quantize_act(xd)
        del xd
        wq, sw = w8a8.quantize_weight(_dev_bf16(w, dev))
        b = _dev_bf16(bb, dev)
        row = {"name": s.name, "M": s.M, "N": s.N, "K": s.K, "m_lo": lo, "m_hi": hi,
               "default": w8a8.tile_name(w8a8.default_tile(s.M, s.N, s.K)), "ms": {}}
        y = torch.empty((s.M, s.N), dtype=torch.bfloat16, device=dev)
        nws = max(w8a8.gemm_workspace_bytes(s.M, s.N, s.K, t) for t in range(w8a8.tile_count()))
        ws = torch.empty(max(nws, 1), dtype=torch.uint8, device=dev)
        it = iters if s.ops < 5e14 else max(3, iters // 4)
        def wanted(t):
            name = w8a8.tile_name(t)
            if s.M > 128 and name.startswith(("skinny", "wsx")):
                return False
            d = _tile_dims(name)
            # split-K only pays where the unsplit tiles leave CUs idle
            if "_k" in name and -(-s.M // d[0]) * -(-s.N // d[1]) >= 2 * CUS:
                return False
            return True
        cand = [t for t in range(w8a8.tile_count()) if wanted(t)]
        first = w8a8.select_tile(s.M, s.N, s.K)
        time_ms(lambda: w8a8.gemm(xq, sx, wq, sw, b, tile=first, out=y, workspace=ws), it,
                warm_ms=30.0)
        for _ in range(2):
            for t in cand:
                name = w8a8.tile_name(t)
                ms = time_ms(lambda: w8a8.gemm(xq, sx, wq, sw, b, tile=t, out=y, workspace=ws),
                             it)
                row["ms"][name] = min(ms, row["ms"].get(name, ms))
        best = min(row["ms"], key=row["ms"].get)
        row["best"] = best
        row["best_tops"] = 2 * s.M * s.N * s.K / (row["ms"][best] * 1e-3) / 1e12
        print(json.dumps(row), flush=True)
        results.append(row)
        del xq, sx, wq, sw, b, y, ws
        torch.cuda.empty_cache()
    return results


def _tile_dims(name):
    m = re.match(r"m(\d+)n(\d+)k(\d+)", name)
    return tuple(int(g) for g in m.groups()) if m else None


# ---------------------------------------------------------------- cost models

# The register-staged tiles, which were never the fastest, stay out of the models.
UNMODELED = {"m128n128k128w2x2", "m64n128k128w1x4", "m32n128k128w1x4", "m32n64k128w1x2"}


def random_shape(rng, m_max=8192):
    """M 17..m_max, K 256..24576 and N 128..20480, log-uniform multiples of 16 (K and N), in
    half of the shapes of 256 and 128, up to 5e11 int8 ops."""
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    while True:
        M, K, N = log(17, m_max), log(256, 24576), log(128, 20480)
        wide = rng.random() < 0.5
        K, N = (K // 256 * 256, N // 128 * 128) if wide else (K // 16 * 16, N // 16 * 16)
        if 2.0 * M * N * K < 5e11 and N * K < 340_000_000:
            return M, N, K


def sweep_random(n, seed, m_max):
    """us of every modeled tile and of the default plan on n random shapes, the weights taken
    in turn from 700 MB (from HBM, as a program of many layers has them)."""
    dev = torch.device("cuda:0")
    rng = random.Random(seed)
    gen = torch.Generator(device=dev).manual_seed(seed)
    names = [w8a8.tile_name(t) for t in range(w8a8.tile_count())]
    pool = torch.empty(700_000_000, dtype=torch.int8, device=dev)
    for part in pool.split(100_000_000):
        part.copy_((33 * torch.randn(part.numel(), device=dev, generator=gen)).clamp_(-127, 127))
    rows = []
    for i in range(n):
        M, N, K = random_shape(rng, m_max)
        copies = max(1, min(20, pool.numel() // (N * K)))
        wqs = [pool[j * N * K:(j + 1) * N * K].view(N, K) for j in range(copies)]
        xq = (10 * torch.randn(M, K, device=dev, generator=gen)).clamp_(-127, 127).to(torch.int8)
        sx, sw = torch.rand(M, device=dev) * 0.01, torch.rand(N, device=dev) * 0.01
        y = torch.empty((M, N), dtype=torch.bfloat16, device=dev)
        cand = [t for t, name in enumerate(names) if name not in UNMODELED and
                (_tile_dims(name) or M <= 128)]
        ws = torch.empty(max(1, *(w8a8.gemm_workspace_bytes(M, N, K, t) for t in [-1] + cand)),
                         dtype=torch.uint8, device=dev)
        row = {"M": M, "N": N, "K": K, "plan": w8a8.plan_name(M, N, K),
               "fallback": w8a8.tile_name(w8a8.default_tile(M, N, K)), "us": {}}

        def timed(t, warm):
            def calls():
                for wq in wqs:
                    w8a8.gemm(xq, sx, wq, sw, tile=t, out=y, workspace=ws)
            return round(1e3 * time_ms(calls, 1, 1, warm, 1.5) / copies, 3)
        timed(-1, 5.0)
        for t in [-1] + cand:
            row["us"]["plan" if t < 0 else names[t]] = timed(t, 0.0)
        rows.append(row)
        if i % 50 == 49:
            print(f"{i + 1} of {n} shapes", flush=True)
    return rows


def _cdiv(a, b):
    return -(-a // b)


def _stream_dims(name):
    m = re.match(r"(skinny|wsx)_m(\d+)n(\d+)w(\d+)", name)
    return (m[1] == "wsx", *(int(g) for g in m.groups()[1:])) if m else None


def stream_fits(name, M, K):
    """Whether a streaming tile runs its own kernel: the token block of a wsx tile has to fit
    in LDS (wsx_lds_bytes in gemm_i8.hip), else the register-staged kernel of its shape runs."""
    wsx, tm, tn, nw = _stream_dims(name)
    body = max(min(M, tm) * (_cdiv(K, 1024) * 1024 + 16), nw * (tn // 16) * (tm // 16) * 1024)
    return not wsx or _cdiv(64 * (tm // 16) + 4 * nw, 256) * 256 + body <= 160 * 1024


def cost_terms(name, M, N, K):
    """What the tile's cost is linear in: (c, d) of kTileCost, or the eight of kStreamCost."""
    d = _tile_dims(name)
    if d:
        rounds = _cdiv(_cdiv(M, d[0]) * _cdiv(N, d[1]), CUS)
        return [1e3 * rounds, 1e-6 * rounds * K * d[0] * d[1]]
    _, tm, tn, _ = _stream_dims(name)
    wgs = _cdiv(M, tm) * _cdiv(N, tn)
    more = _cdiv(wgs, CUS) - 1
    return [1.0, 1e-3 * K, more, 1e-3 * more * K, 1e-6 * wgs * K * tn,
            1e-6 * wgs * K * min(M, tm), 1e-6 * N * K, 1e-3 * K * (K % 256 == 0)]


def fit_costs(rows, names):
    """Coefficients by tile: least squares on the relative error with coefficients >= 0,
    each shape weighed by how near the tile is to the fastest one there (a tile's time
    matters where it may be chosen)."""
    out = {}
    for name in names:
        if name in UNMODELED or re.search(r"_k\d+$", name):
            continue
        use = [r for r in rows if name in r["us"] and
               (_tile_dims(name) or stream_fits(name, r["M"], r["K"]))]
        w = np.array([(min(r["us"].values()) / r["us"][name]) ** 2 for r in use])
        a = np.array([cost_terms(name, r["M"], r["N"], r["K"]) for r in use])
        a = a * (w / np.array([r["us"][name] for r in use]))[:, None]
        keep = list(range(a.shape[1]))
        while True:
            x = np.linalg.lstsq(a[:, keep], w, rcond=None)[0]
            if (x >= 0).all():
                break
            keep = [k for k, v in zip(keep, x) if v > 0]
        out[name] = np.zeros(a.shape[1])
        out[name][keep] = x
    return out


def fit_split(rows, names, costs):
    """(fixed, per K-range, per MB of partials) us of a split besides its main launch, from
    the tiles whose name ends in _k<s>."""
    a, y = [], []
    for name in names:
        m = re.match(r"(.*)_k(\d+)$", name)
        if not m or m[1] not in costs:
            continue
        bk = _tile_dims(m[1])[2]
        for r in (r for r in rows if name in r["us"]):
            per = _cdiv(_cdiv(r["K"], bk), int(m[2])) * bk
            n = _cdiv(r["K"], per)
            if n == 1:
                continue
            M, N = r["M"], r["N"]
            d = _tile_dims(m[1])
            rounds = _cdiv(_cdiv(M, d[0]) * _cdiv(N, d[1]) * n, CUS)
            main = np.dot(costs[m[1]], [1e3 * rounds, 1e-6 * rounds * per * d[0] * d[1]])
            a.append(np.array([1.0, n, 4e-6 * n * M * N]) / r["us"][name])
            y.append(1.0 - main / r["us"][name])
    return np.linalg.lstsq(np.array(a), np.array(y), rcond=None)[0]


def report_fit(rows, names):
    costs = fit_costs(rows, names)
    print("split K, us: fixed %.2f, per range %.3f, per MB %.3f" % tuple(fit_split(rows, names, costs)))
    print("kTileCost:")
    for name in names:
        c = costs.get(name, (0.0, 0.0)) if _tile_dims(name) else (0.0, 0.0)
        print(f"    {{{c[0]:.6e}, {c[1]:.6e}}},  // {name}")
    print("kStreamCost:")
    for i, name in enumerate(names):
        if _stream_dims(name):
            print(f"    {{{i}, " + ", ".join(f"{v:.4f}" for v in costs[name]) + f"}},  // {name}")

    def mean(v):
        return math.exp(sum(map(math.log, v)) / len(v))
    for lo, hi in ((17, 32), (33, 64), (65, 128), (129, 512), (513, 8192)):
        use = [r for r in rows if lo <= r["M"] <= hi]
        if not use:
            continue
        best = [min(r["us"].values()) for r in use]
        for what, us in (("default plan", [r["us"]["plan"] for r in use]),
                         ("fallback tile", [r["us"].get(r["fallback"], r["us"]["plan"])
                                            for r in use])):
            over = [u / b for u, b in zip(us, best)]
            print(f"M {lo}..{hi}, {len(use)} shapes: {what} over the fastest "
                  f"{mean(over):.3f} (geometric mean), worst {max(over):.2f}")


def write_table(results, path):
    names = [w8a8.tile_name(t) for t in range(w8a8.tile_count())]
    # the cost models are fitted to random shapes, not to these: they stay as they are
    old = open(os.path.join(os.path.dirname(os.path.abspath(__file__)), "csrc",
                            "tile_table.inc")).read()
    costs = old[old.index("// Cost model per tile"):old.index("static const TableEntry")]
    lines = [HEADER, costs.rstrip(), ""]
    lines.append("static const TableEntry kTileTable[] = {")
    for r in results:
        lines.append(f"    {{{r['m_lo']}, {r['m_hi']}, {r['N']}, {r['K']}, "
                     f"{names.index(r['best'])}}},  // M={r['M']} {r['best']} "
                     f"{r['best_tops']:.0f} TOPS")
    lines.append("    {0, 0, 0, 0, -1},  // sentinel")
    lines.append("};")
    with open(path, "w") as f:
        f.write("\n".join(lines) + "\n")


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--out")
    ap.add_argument("--json")
    ap.add_argument("--iters", type=int, default=20)
    ap.add_argument("--set", default="all", choices=["all", "workloads", "paper"])
    ap.add_argument("--from-json", help="rewrite the table from a saved sweep (no timing)")
    ap.add_argument("--random", type=int, help="time this many random shapes into --json")
    ap.add_argument("--seed", type=int, default=1)
    ap.add_argument("--m-max", type=int, default=8192)
    ap.add_argument("--fit", nargs="+", help="fit the cost models to saved random sweeps")
    a = ap.parse_args()
    if a.fit:
        rows = []
        for path in a.fit:
            with open(path) as f:
                rows += json.load(f)
        report_fit(rows, [w8a8.tile_name(t) for t in range(w8a8.tile_count())])
        return
    if a.random:
        if not a.json:
            ap.error("--random needs --json")
        with open(a.json, "w") as f:
            json.dump(sweep_random(a.random, a.seed, a.m_max), f)
        return
    if not a.out:
        ap.error("--out is needed")
    if a.from_json:
        with open(a.from_json) as f:
            res = json.load(f)
        for r in res:
            r.setdefault("m_lo", r["M"])
            r.setdefault("m_hi", r["M"])
    else:
        res = sweep(a.iters, a.set)
    write_table(res, a.out)
    if a.json and not a.from_json:
        with open(a.json, "w") as f:
            json.dump(res, f, indent=1)


if __name__ == "__main__":
    main()
