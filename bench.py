"""Benchmark of the fused W8A8 linear on one MI355X.

One step is one pass of the hot path over one batch: for each linear, per-token int8
quantization of the activations, then the int8 GEMM with the fused dequantization + bias
epilogue (the weights are quantized once, before timing: an offline step). The workload
is the four linears of a DiT block at a 1024px-like sequence, M = 4608 tokens (4096
image + 512 text): qkv (K = 4096, N = 12288), attention out (4096, 4096), MLP up (4096,
16384) and MLP down (16384, 4096), on seeded synthetic bf16 inputs; value = the four
linears' 2MNK / step time. Before the W warm-up steps the step runs untimed for 60 ms:
under sustained int8 MFMA load the chip's clocks dip for ~15 ms after a start or an idle
gap before they settle.

Prints one JSON line. Besides the required fields it carries:
  roofline      the dominant kernel (the GEMM with the longest launch) and its achieved
                int8 ops/s (2MNK per launch / its mean HIP-event duration, launched back
                to back on the benchmark stream) against MI355X's dense int8 peak;
                traffic = HBM bytes per launch from rocprofv3 counters when they were
                taken on the current kernel source, else null; mfma_ceiling = what the
                int8 matrix cores sustain on this GEMM's own codes (its MFMA sequence
                replayed from registers), against which the GEMM's rate is also given
  shapes        per linear: tile (with its K split), GEMM and quantizer durations, and (full run) the whole
                linear with bf16 / fake-quant / unfused-int8 comparators
  comparators   the same comparators summed over one step
  config1_attn_proj  the 768px attention projection (M = 2560, K = N = 4096) alone
  cpu_baseline  the CPU oracle timed on this host over a bounded row sample of the step
  health_gate   bf16 GEMM TFLOP/s of this card (the paper's bf16 health check idea)

Usage: python bench.py [--gpus 1] [--steps K] [--warmup W] [--no-cpu] [--no-extra]
       python bench.py --all-shapes           (every workload shape, one JSON line each)
       python bench.py --recipe               (GELU / SmoothQuant quantizer, shared X)
       python bench.py --paper-shapes         (the paper's five shapes, as shipped and untuned)
       python bench.py --gemm-study           (headline GEMMs on other operand bits, hipBLASLt int8)
       python bench.py --copy-calibration     (a known-size copy for counter scaling)
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import re
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

# MI355X published dense peaks (no sparsity): int8 5.0 POP/s is 256 CU x 2.4 GHz x 8192
# int8 ops/clk/CU = 5033.2 TOP/s; HBM3E 8 TB/s; bf16 2516.6 TFLOP/s.
PEAK_INT8_TOPS = 256 * 2.4e9 * 8192 / 1e12
PEAK_BF16_TFLOPS = PEAK_INT8_TOPS / 2
PEAK_HBM_GBS = 8000.0
HEALTH_MIN_BF16_TFLOPS = 600.0

# The headline workload: the four linears of a DiT block at a 1024px-like sequence,
# M = 4608 tokens (4096 image + 512 text), hidden size 4096, with per-token quantization
# in the timed path. One step runs all four through w8a8_linear.
HEADLINE_CONFIG = 3
HEADLINE_NAMES = ("qkv", "attn_out", "mlp_up", "mlp_down")
# Kept beside it: the 768px attention projection (M = 2560, K = N = 4096).
SECOND = dict(name="attn_proj", config=1)

GEMM_SRC = [os.path.join(ROOT, "paper_2606_14598_amd", "csrc", f)
            for f in ("gemm_i8.hip", "tile_table.inc", "w8a8_internal.hpp")]
PROFILES = os.path.join(ROOT, "profiles")
# Time-based settle before the warm-up steps: the chip's clocks settle only after
# ~15-20 ms of sustained int8 MFMA load.
SETTLE_MS = 60.0


def counters_file(name: str, M: int, N: int, K: int) -> str:
    return os.path.join(PROFILES, f"gemm_{name}_m{M}_n{N}_k{K}_counters.md")


# ------------------------------------------------------------------ byte/op models

def gemm_ops(M: int, N: int, K: int) -> int:
    return 2 * M * N * K


def gemm_bytes(M: int, N: int, K: int, with_vectors: bool = True) -> int:
    """Algorithmic HBM bytes of the fused GEMM: int8 X [M,K] and W [N,K] read once, bf16
    Y [M,N] written once; with_vectors adds the fp32 scales sx [M], sw [N] and the bf16
    bias [N]. Without them this is the paper's roofline byte count (int8 operands, bf16
    output), which reproduces its 768..6337 ops/byte range."""
    b = M * K + N * K + 2 * M * N
    if with_vectors:
        b += 4 * M + 4 * N + 2 * N
    return b


def quant_bytes(M: int, K: int) -> int:
    """Per-token quantizer: bf16 X read, int8 Xq written, fp32 sx written."""
    return 3 * M * K + 4 * M


def _code_only(text: str) -> str:
    """C++ source without comments and blank space, so that a comment edit does not
    count as a kernel change (string literals here hold no comment markers)."""
    text = re.sub(r"/\*.*?\*/", " ", text, flags=re.S)
    text = re.sub(r"//[^\n]*", " ", text)
    return " ".join(text.split())


def gemm_source_hash() -> str:
    """Identity of the GEMM kernel code (comments and whitespace ignored): the stored
    HBM-traffic counters apply only while it is unchanged."""
    h = hashlib.sha256()
    for p in GEMM_SRC:
        with open(p, encoding="utf-8") as f:
            h.update(_code_only(f.read()).encode())
    return h.hexdigest()[:16]


def stored_traffic(path: str):
    """HBM bytes per GEMM launch from a committed counter summary, if it was taken on
    the current GEMM source."""
    try:
        text = open(path).read()
    except OSError:
        return None
    src = re.search(r"gemm_source_sha256_16:\s*([0-9a-f]+)", text)
    tb = re.search(r"traffic_bytes_per_launch:\s*([0-9.e+]+)", text)
    if not src or not tb or src.group(1) != gemm_source_hash():
        return None
    return float(tb.group(1))


# ------------------------------------------------------------------ helpers

def dev_bf16(bits, dev):
    import numpy as np
    import torch
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).view(torch.bfloat16).to(dev)


def time_loop(fn, iters: int, warmup: int = 3) -> float:
    """Mean ms per call of fn over `iters` calls, HIP events on the current stream."""
    import torch
    for _ in range(warmup):
        fn()
    s, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    s.record()
    for _ in range(iters):
        fn()
    e.record()
    torch.cuda.synchronize()
    return s.elapsed_time(e) / iters


def health_gate(dev) -> dict:
    import torch
    n = 8192
    a = torch.randn(n, n, device=dev, dtype=torch.bfloat16)
    b = torch.randn(n, n, device=dev, dtype=torch.bfloat16)
    ms = time_loop(lambda: torch.matmul(a, b), 10, warmup=3)
    tf = 2 * n ** 3 / (ms * 1e-3) / 1e12
    del a, b
    return {"bf16_gemm_8192_tflops": round(tf, 1), "threshold": HEALTH_MIN_BF16_TFLOPS,
            "pass": tf >= HEALTH_MIN_BF16_TFLOPS, "smi": smi_snapshot()}


def time_weight_quant(wd, iters=10):
    import paper_2606_14598_amd as w8a8
    return time_loop(lambda: w8a8.quantize_weight(wd), iters)


def comparators(shp, xd, wd, bd, wq, sw, iters):
    """bf16 F.linear, the fake-quant path and the unfused int8 path on the same inputs."""
    import torch
    import torch.nn.functional as F
    out = {}
    out["bf16_linear_ms"] = time_loop(lambda: F.linear(xd, wd, bd), iters)

    def fake_quant():
        # Dequantize-to-bf16 then bf16 matmul: W8A8 codes round-tripped through bf16.
        wdq = (wq.to(torch.float32) * sw[:, None]).to(torch.bfloat16)
        xf = xd.to(torch.float32)
        a = xf.abs().amax(dim=1, keepdim=True)
        s = a / 127.0
        q = torch.clamp(torch.round(xf * (127.0 / a)), -127, 127)
        xdq = (q * s).to(torch.bfloat16)
        return F.linear(xdq, wdq, bd)
    out["fake_quant_ms"] = time_loop(fake_quant, iters)

    import paper_2606_14598_amd as w8a8
    xq, sx = w8a8.quantize_act(xd)
    try:
        wt = wq.t().contiguous()
        torch._int_mm(xq, wt)

        def unfused():
            acc = torch._int_mm(xq, wt)
            return (acc.to(torch.float32) * (sx[:, None] * sw[None, :]) +
                    bd.to(torch.float32)).to(torch.bfloat16)
        out["unfused_int8_ms"] = time_loop(unfused, iters)
        out["unfused_int8_gemm"] = "torch._int_mm + torch dequant"
    except Exception:  # noqa: BLE001
        def unfused():
            acc = w8a8.gemm_acc_i32(xq, wq)
            return (acc.to(torch.float32) * (sx[:, None] * sw[None, :]) +
                    bd.to(torch.float32)).to(torch.bfloat16)
        out["unfused_int8_ms"] = time_loop(unfused, iters)
        out["unfused_int8_gemm"] = "w8a8_gemm_acc_i32 + torch dequant"
    return {k: (round(v, 4) if isinstance(v, float) else v) for k, v in out.items()}


def single_thread_tiny_ms() -> float:
    """The oracle on one thread over the tiny workload (64 x 256 x 128), for scale."""
    import oracle
    import synth_inputs as si
    threads = oracle.max_threads()
    x0, w0, b0 = si.make_inputs(si.workload(0, "tiny"))
    wq0, sw0 = oracle.quantize_rows(w0, nthreads=1)
    t0 = time.perf_counter()
    n1 = 0
    while time.perf_counter() - t0 < 0.5:
        oracle.linear(x0, wq0, sw0, b0, nthreads=1)
        n1 += 1
    t1 = (time.perf_counter() - t0) / n1
    oracle.quantize_rows(w0[:1], nthreads=threads)   # the thread setting is process-wide
    return round(t1 * 1e3, 3)


def cpu_model() -> str:
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def gfx_clock_mhz(data) -> list:
    """Current gfx clocks (MHz) found in an amd-smi metric --clock JSON document."""
    out = []
    def walk(o, key=""):
        if isinstance(o, dict):
            if key.startswith("gfx") and isinstance(o.get("clk"), dict):
                v = o["clk"].get("value")
                if isinstance(v, (int, float)):
                    out.append(float(v))
            for k, v in o.items():
                walk(v, str(k))
        elif isinstance(o, list):
            for v in o:
                walk(v, key)
    walk(data)
    return out


def clock_under_load(fn, seconds: float = 3.0) -> dict:
    """The gfx clock while fn runs back to back: amd-smi is polled from a host thread
    while the GPU stays busy; the mean over polls and engines is reported."""
    import subprocess
    import threading
    import torch
    samples, errors = [], []

    def poll():
        for _ in range(3):
            try:
                r = subprocess.run(["amd-smi", "metric", "-g", "0", "--clock", "--json"],
                                   capture_output=True, text=True, timeout=20)
                if r.returncode == 0:
                    samples.extend(gfx_clock_mhz(json.loads(r.stdout)))
                else:
                    errors.append((r.stderr or r.stdout).strip()[:120])
            except Exception as e:  # noqa: BLE001 -- a measurement aid, never fatal
                errors.append(f"{type(e).__name__}: {e}"[:120])
    th = threading.Thread(target=poll)
    t0 = time.perf_counter()
    th.start()
    while th.is_alive() and time.perf_counter() - t0 < 60:
        for _ in range(200):
            fn()
        torch.cuda.synchronize()
    th.join(timeout=60)
    if not samples:
        return {"error": errors[0] if errors else "no gfx clock in amd-smi output"}
    return {"gfx_mhz_mean": round(sum(samples) / len(samples), 1),
            "gfx_mhz_min": min(samples), "gfx_mhz_max": max(samples),
            "samples": len(samples), "source": "amd-smi metric --clock (reported gfx clock)"}


def mfma_ceiling(w8a8, xq, wq, gemm_tops: float, iters: int = 800, warm_ms: float = 30.0,
                 n: int = 10) -> dict:
    """The int8 matrix-core ceiling on this workload's own codes: the GEMM's per-K-step
    MFMA sequence replayed from registers (w8a8_mfma_ceiling), warmed by time, then n
    launches between HIP events."""
    import time
    import torch
    sums = torch.empty(1024, dtype=torch.int32, device=xq.device)

    def f():
        w8a8.mfma_ceiling(xq, wq, iters, out=sums)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    while (time.perf_counter() - t0) * 1e3 < warm_ms:
        f()
        torch.cuda.synchronize()
    ms = time_loop(f, n, warmup=0)
    tops = w8a8.mfma_ceiling_ops(iters) / (ms * 1e-3) / 1e12
    return {"tops": round(tops, 1), "frac_of_peak": round(tops / PEAK_INT8_TOPS, 4),
            "gemm_frac_of_ceiling": round(gemm_tops / tops, 4),
            "what": "the GEMM's MFMA sequence (per wavefront and K-step, 2 weight x 5 token "
                    "fragments of v_mfma_i32_32x32x32_i8) replayed from registers on this "
                    "workload's Xq/Wq fragments, no memory traffic (w8a8_mfma_ceiling)"}


def smi_snapshot() -> dict:
    """Clocks and temperature of GPU 0 as amd-smi reports them (read-only query, bounded
    by a timeout); an error string if the tool is missing or fails."""
    import subprocess
    try:
        r = subprocess.run(["amd-smi", "metric", "-g", "0", "--clock", "--temperature",
                            "--json"], capture_output=True, text=True, timeout=20)
        if r.returncode != 0:
            return {"error": (r.stderr or r.stdout).strip()[:200]}
        data = json.loads(r.stdout)
        return {"amd_smi": data if len(r.stdout) < 4000 else r.stdout[:4000]}
    except Exception as e:  # noqa: BLE001 -- a snapshot must never fail the benchmark
        return {"error": f"{type(e).__name__}: {e}"[:200]}


# ------------------------------------------------------------------ main measurement

class Linear:
    """One workload linear on the device: inputs, quantized weight, output, workspace and
    the raw ctypes arguments of its w8a8_linear / quantize / GEMM calls."""

    def __init__(self, shp, dev, lib):
        import ctypes
        import torch
        import paper_2606_14598_amd as w8a8
        self.shp = shp
        M, N, K = shp.M, shp.N, shp.K
        self.x, self.w, self.b = __import__("synth_inputs").make_inputs(shp)
        self.xd, self.wd, self.bd = (dev_bf16(t, dev) for t in (self.x, self.w, self.b))
        self.wq, self.sw = w8a8.quantize_weight(self.wd)
        self.xq = torch.empty((M, K), dtype=torch.int8, device=dev)
        self.sx = torch.empty((M,), dtype=torch.float32, device=dev)
        self.y = torch.empty((M, N), dtype=torch.bfloat16, device=dev)
        self.gws = torch.empty(max(1, w8a8.gemm_workspace_bytes(M, N, K)), dtype=torch.uint8,
                               device=dev)
        self.lws = torch.empty(w8a8.linear_workspace_bytes(M, N, K), dtype=torch.uint8,
                               device=dev)
        self.tile_name = w8a8.plan_name(M, N, K)
        self.lib = lib
        P = ctypes.c_void_p
        self.a = {k: P(getattr(self, k).data_ptr())
                  for k in ("xd", "xq", "sx", "wq", "sw", "bd", "y", "gws", "lws")}

    def linear(self, sp):
        a, s = self.a, self.shp
        st = self.lib.w8a8_linear(a["xd"], a["wq"], a["sw"], a["bd"], a["y"], s.M, s.N, s.K,
                                  a["lws"], self.lws.numel(), sp)
        if st:
            raise RuntimeError(f"w8a8_linear status {st}")

    def quant(self, sp):
        a, s = self.a, self.shp
        st = self.lib.w8a8_quantize_act(a["xd"], s.M, s.K, a["xq"], a["sx"], sp)
        if st:
            raise RuntimeError(f"w8a8_quantize_act status {st}")

    def gemm(self, sp):
        a, s = self.a, self.shp
        st = self.lib.w8a8_gemm(a["xq"], a["sx"], a["wq"], a["sw"], a["bd"], a["y"], s.M,
                                s.N, s.K, a["gws"], self.gws.numel(), sp)
        if st:
            raise RuntimeError(f"w8a8_gemm status {st}")

    @property
    def ops(self):
        return gemm_ops(self.shp.M, self.shp.N, self.shp.K)


def run(args) -> dict:
    import ctypes
    import torch
    import paper_2606_14598_amd as w8a8
    import synth_inputs as si
    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    lib = w8a8.load_library()

    health = health_gate(dev) if not args.no_extra else None

    lins = [Linear(si.workload(HEADLINE_CONFIG, n), dev, lib) for n in HEADLINE_NAMES]
    stream = torch.cuda.current_stream(dev)
    sp = ctypes.c_void_p(stream.cuda_stream)

    def step():
        # One pass of the hot path over the block's four linears: per-token quantizer +
        # fused int8 GEMM/epilogue each, through the product entry point.
        for L in lins:
            L.linear(sp)

    def timed(fn, n):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        start.record(stream)
        for _ in range(n):
            fn()
        end.record(stream)
        torch.cuda.synchronize()
        return start.elapsed_time(end) / n

    # Untimed: a time-based settle, then the W warm-up steps, then exactly K timed steps.
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    while (time.perf_counter() - t0) * 1e3 < SETTLE_MS:
        step()
        torch.cuda.synchronize()
    for _ in range(args.warmup):
        step()
    ms_step = timed(step, args.steps)

    # Per-kernel mean durations: each linear's GEMM and quantizer launched back to back on
    # the benchmark stream, HIP events around the loop.
    per = []
    for L in lins:
        L.quant(sp)
        gms = timed(lambda: L.gemm(sp), args.steps)
        qms = timed(lambda: L.quant(sp), args.steps)
        per.append((gms, qms))
    # The dominant kernel: the GEMM with the longest launch.
    dom = max(range(len(lins)), key=lambda i: per[i][0])
    D = lins[dom]
    gemm_ms = per[dom][0]
    ops_step = sum(L.ops for L in lins)
    value_tops = ops_step / (ms_step * 1e-3) / 1e12
    gemm_tops = D.ops / (gemm_ms * 1e-3) / 1e12
    Ds = D.shp
    traffic = stored_traffic(counters_file(Ds.name, Ds.M, Ds.N, Ds.K))

    shapes_desc = ", ".join(f"{L.shp.name} K={L.shp.K} N={L.shp.N}" for L in lins)
    rec = {
        "metric": "INT8 TOPS per GEMM shape, % of dense INT8 MFMA peak, speedup vs bf16 GEMM",
        "value": round(value_tops, 2),
        "unit": "TOPS",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_step, 5),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "i8",
        "data": "synthetic",
        "config": {"workload": f"DiT block GEMMs at a 1024px-like sequence: M={lins[0].shp.M} "
                               f"tokens (4096 image + 512 text), the four W8A8 linears "
                               f"{shapes_desc}, bf16 in/out with bias, per-token "
                               f"quantization in the timed path",
                   "M": lins[0].shp.M,
                   "linears": [{"name": L.shp.name, "K": L.shp.K, "N": L.shp.N,
                                "tile": L.tile_name, "seed": L.shp.seed} for L in lins],
                   "timed": "one step = w8a8_linear (per-token quantizer + fused int8 "
                            "GEMM/epilogue) on each of the four linears; value = sum of "
                            "2MNK over the four / step time",
                   "settle_ms_before_warmup": SETTLE_MS},
        "pct_of_int8_peak": round(100 * value_tops / PEAK_INT8_TOPS, 2),
        "roofline": {"bound": "mfma", "achieved": round(gemm_tops, 2),
                     "peak": round(PEAK_INT8_TOPS, 1), "unit": "TFLOP/s",
                     "frac": round(gemm_tops / PEAK_INT8_TOPS, 4),
                     "traffic": traffic,
                     "kernel": f"gemm_i8 {D.tile_name} on {Ds.name} (M={Ds.M} K={Ds.K} "
                               f"N={Ds.N}; int8 ops counted 2 per MAC)",
                     "gemm_ms": round(gemm_ms, 5),
                     "duration_from": "HIP events around back-to-back launches of this GEMM "
                                      "on the benchmark stream",
                     "algorithmic_bytes": gemm_bytes(Ds.M, Ds.N, Ds.K),
                     "source": gemm_source_hash()},
    }
    per_shape = []
    for L, (gms, qms) in zip(lins, per):
        s = L.shp
        qb = quant_bytes(s.M, s.K)
        per_shape.append({"shape": s.name, "M": s.M, "K": s.K, "N": s.N, "tile": L.tile_name,
                          "gemm_ms": round(gms, 5),
                          "gemm_tops": round(L.ops / gms / 1e9, 1),
                          "gemm_frac_of_peak": round(L.ops / gms / 1e9 / PEAK_INT8_TOPS, 4),
                          "quantizer_ms": round(qms, 5),
                          "quantizer_GB_s": round(qb / (qms * 1e-3) / 1e9, 1)})
    rec["shapes"] = per_shape

    if not args.no_extra:
        rec["health_gate"] = health
        it = max(10, args.steps)
        comp_tot = {"bf16_linear_ms": 0.0, "fake_quant_ms": 0.0, "unfused_int8_ms": 0.0}
        for L, ps in zip(lins, per_shape):
            c = comparators(L.shp, L.xd, L.wd, L.bd, L.wq, L.sw, it)
            for k in comp_tot:
                comp_tot[k] += c[k]
            lin_ms = timed(lambda: L.linear(sp), it)
            ps.update({"linear_ms": round(lin_ms, 5), **c,
                       "speedup_vs_bf16": round(c["bf16_linear_ms"] / lin_ms, 3)})
            comp_tot["unfused_int8_gemm"] = c["unfused_int8_gemm"]
        comp = {k: (round(v, 4) if isinstance(v, float) else v) for k, v in comp_tot.items()}
        comp["speedup_vs_bf16"] = round(comp_tot["bf16_linear_ms"] / ms_step, 3)
        comp["speedup_vs_fake_quant"] = round(comp_tot["fake_quant_ms"] / ms_step, 3)
        comp["speedup_vs_unfused_int8"] = round(comp_tot["unfused_int8_ms"] / ms_step, 3)
        comp["weight_quant_ms"] = round(time_weight_quant(D.wd), 4)
        comp["what"] = "sums over the four linears of one step, same inputs"
        rec["comparators"] = comp
        rec["vs_bf16_gemm"] = comp["speedup_vs_bf16"]
        # the clock the chip holds under the dominant GEMM, and the peak at that clock
        clk = clock_under_load(lambda: D.gemm(sp))
        rec["roofline"]["clock_under_load"] = clk
        if "gfx_mhz_mean" in clk:
            rec["roofline"]["pct_of_peak_at_measured_clock"] = round(
                100 * gemm_tops / (PEAK_INT8_TOPS * clk["gfx_mhz_mean"] / 2400.0), 2)
        # what the matrix cores sustain on these very codes
        D.quant(sp)
        rec["roofline"]["mfma_ceiling"] = mfma_ceiling(w8a8, D.xq, D.wq, gemm_tops)
        rec["config1_attn_proj"] = second_workload(args, dev, lib, timed, sp)
    if not args.no_cpu:
        rec["cpu_baseline"] = cpu_baseline_block([L.shp for L in lins],
                                                 [(L.x, L.w, L.b) for L in lins])
    return rec


def second_workload(args, dev, lib, timed, sp) -> dict:
    """The 768px attention projection (M = 2560, K = N = 4096), one w8a8_linear per step,
    timed the same way as the headline."""
    import synth_inputs as si
    L = Linear(si.workload(SECOND["config"], SECOND["name"]), dev, lib)
    for _ in range(max(args.warmup, 50)):
        L.linear(sp)
    ms = timed(lambda: L.linear(sp), max(args.steps, 50))
    L.quant(sp)
    gms = timed(lambda: L.gemm(sp), max(args.steps, 50))
    s = L.shp
    return {"workload": f"DiT attention projection at a 768px-like sequence: M={s.M}, "
                        f"K={s.K}, N={s.N}", "tile": L.tile_name,
            "linear_ms": round(ms, 5), "linear_tops": round(L.ops / ms / 1e9, 1),
            "gemm_ms": round(gms, 5), "gemm_tops": round(L.ops / gms / 1e9, 1),
            "gemm_frac_of_peak": round(L.ops / gms / 1e9 / PEAK_INT8_TOPS, 4)}


def cpu_baseline_block(shapes, inputs, budget_s: float = 12.0) -> dict:
    """The CPU oracle (as it stands) on a bounded sample of the headline step: the same
    number of token rows of each of the four linears (per-token quantization, exact
    integer product, epilogue against the full weight), repeated until about budget_s
    seconds have passed. Reported in the metric's unit (int8 TOP/s)."""
    import numpy as np
    import oracle
    threads = oracle.max_threads()
    wqs = [oracle.quantize_rows(w) for (_, w, _) in inputs]
    rows = threads

    def one_pass(r):
        for (x, _, b), (wq, sw) in zip(inputs, wqs):
            oracle.linear(np.ascontiguousarray(x[:r]), wq, sw, b)

    t0 = time.perf_counter()
    one_pass(rows)
    t = time.perf_counter() - t0
    rows = int(min(shapes[0].M, max(rows, rows * (budget_s / 3) / max(t, 1e-3))))
    rows = max(threads, rows // threads * threads)
    reps, total = 0, 0.0
    while total < budget_s and reps < 1000:
        t0 = time.perf_counter()
        one_pass(rows)
        total += time.perf_counter() - t0
        reps += 1
    ops = sum(gemm_ops(rows, s.N, s.K) for s in shapes) * reps
    return {"value": round(ops / total / 1e12, 6), "unit": "TOPS", "cores": threads,
            "kind": "oracle",
            "sample": f"{reps} x {rows} of {shapes[0].M} token rows of each of the four "
                      f"linears (quantize + int8 product + epilogue against the full "
                      f"weights), {total:.1f} s",
            "cpu_model": cpu_model(),
            "single_thread_tiny_ms": single_thread_tiny_ms()}


FIXED_TILE = 0   # one configuration for every shape: the untuned-by-design arm


def graph_ms(fn, iters: int = 20, warm_ms: float = 25.0, min_timed_ms: float = 3.0) -> float:
    """Mean ms per call of fn: `iters` calls captured in one HIP graph (no host launch
    overhead in the measurement, which matters for microsecond shapes), replayed until
    `warm_ms` of sustained work has run (the power management of the chip settles only
    after ~15-20 ms of load), then timed over enough replays to cover `min_timed_ms`."""
    import torch
    for _ in range(3):
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
    for _ in range(int(warm_ms / once) + 1):
        g.replay()
    reps = max(3, int(min_timed_ms / once) + 1)
    torch.cuda.synchronize()
    st.record()
    for _ in range(reps):
        g.replay()
    en.record()
    torch.cuda.synchronize()
    return st.elapsed_time(en) / (reps * iters)


def all_shapes(args):
    """Every workload shape through the product path (w8a8_linear: per-token quantizer +
    fused GEMM), plus the fused GEMM alone and bf16 F.linear on the same inputs; one JSON
    line per shape."""
    import torch
    import torch.nn.functional as F
    import paper_2606_14598_amd as w8a8
    import synth_inputs as si
    dev = torch.device("cuda:0")
    for cfg in sorted(si.WORKLOADS):
        for shp in si.WORKLOADS[cfg]:
            x, w, b = si.make_inputs(shp)
            xd, wd, bd = dev_bf16(x, dev), dev_bf16(w, dev), dev_bf16(b, dev)
            wq, sw = w8a8.quantize_weight(wd)
            xq, sx = w8a8.quantize_act(xd)
            M, N, K = shp.M, shp.N, shp.K
            y = torch.empty((M, N), dtype=torch.bfloat16, device=dev)
            ws = torch.empty(w8a8.linear_workspace_bytes(M, N, K), dtype=torch.uint8,
                             device=dev)
            gws = torch.empty(max(1, w8a8.gemm_workspace_bytes(M, N, K)), dtype=torch.uint8,
                              device=dev)
            reps = {"lin": [], "gem": [], "bf": []}
            for _ in range(5):
                reps["lin"].append(graph_ms(lambda: w8a8.linear(xd, wq, sw, bd, out=y,
                                                                workspace=ws)))
                reps["gem"].append(graph_ms(lambda: w8a8.gemm(xq, sx, wq, sw, bd, out=y,
                                                              workspace=gws)))
                reps["bf"].append(graph_ms(lambda: F.linear(xd, wd, bd)))
            lin, gem, bf = (sorted(reps[k])[2] for k in ("lin", "gem", "bf"))
            ops = gemm_ops(M, N, K)
            gb = gemm_bytes(M, N, K)
            rec = {"config": cfg, "shape": shp.name, "M": M, "K": K, "N": N,
                   "tile": w8a8.plan_name(M, N, K),
                   "linear_us": round(lin * 1e3, 2), "gemm_us": round(gem * 1e3, 2),
                   "bf16_linear_us": round(bf * 1e3, 2),
                   "linear_tops": round(ops / lin / 1e9, 1),
                   "gemm_tops": round(ops / gem / 1e9, 1),
                   "gemm_pct_int8_peak": round(100 * ops / gem / 1e9 / PEAK_INT8_TOPS, 2),
                   "gemm_hbm_GB_s": round(gb / gem / 1e6, 1),
                   "gemm_pct_hbm": round(100 * gb / gem / 1e6 / PEAK_HBM_GBS, 2),
                   "bound": "mfma" if ops / gb > PEAK_INT8_TOPS * 1e3 / PEAK_HBM_GBS else "hbm",
                   "speedup_linear_vs_bf16": round(bf / lin, 3),
                   "timing": "median of 5 repeats"}
            if M <= 333:
                fns = {"lin": lambda: w8a8.linear(xd, wq, sw, bd, out=y, workspace=ws),
                       "gem": lambda: w8a8.gemm(xq, sx, wq, sw, bd, out=y, workspace=gws),
                       "bf": lambda: F.linear(xd, wd, bd)}
                # Cold (read scrub): each call preceded by a 1 GiB read of another buffer, so
                # the 256 MB MALL holds none of the operands and no dirty lines; in one HIP
                # graph of 10 (scrub, call) pairs, minus the graph of the 10 scrubs alone.
                # This is the call's own time plus one kernel boundary, with no host
                # launch or event-timing floor.
                scrub = torch.zeros((1 << 29) // 4096, 4096, dtype=torch.bfloat16, device=dev)
                amax = torch.empty(4096, dtype=torch.float32, device=dev)
                rs = lambda: w8a8.col_absmax(scrub, out=amax)
                base = graph_ms(rs, iters=10, warm_ms=5.0)
                cold = {k: graph_ms(lambda f=f: (rs(), f()), iters=10, warm_ms=5.0) - base
                        for k, f in fns.items()}
                rec["cold_read_us"] = {"linear": round(cold["lin"] * 1e3, 2),
                                       "gemm": round(cold["gem"] * 1e3, 2),
                                       "bf16_linear": round(cold["bf"] * 1e3, 2)}
                rec["cold_read_gemm_hbm_GB_s"] = round(gb / cold["gem"] / 1e6, 1)
                # The achievable floor: a plain streaming read of Wq's own bytes, timed
                # cold the same way (w8a8_read_ceiling). A weight-streaming GEMM reads
                # those bytes once, so this is the rate HBM actually gives it.
                if wq.numel() % (16 * w8a8.READ_BLOCKS) == 0:
                    rsum = torch.empty(w8a8.READ_BLOCKS, dtype=torch.int32, device=dev)
                    rd = lambda: w8a8.read_ceiling(wq, out=rsum)
                    floor = graph_ms(lambda: (rs(), rd()), iters=10, warm_ms=5.0) - base
                    rec["cold_read_floor_us"] = round(floor * 1e3, 2)
                    rec["cold_read_floor_GB_s"] = round(wq.numel() / floor / 1e6, 1)
                    rec["gemm_cold_frac_of_read_floor"] = round(floor / cold["gem"], 3)
                # Cold (write scrub, the earlier method): a 512 MB scrub write before every
                # call, each call timed alone with HIP events. The scrub leaves the MALL
                # full of dirty lines that the call then writes back, and single-call event
                # timing adds ~6 us of launch floor.
                wscrub = scrub.view(torch.uint8)[: 512 << 20]
                coldw = {"lin": [], "gem": [], "bf": []}
                for _ in range(10):
                    for k, f in fns.items():
                        wscrub.fill_(1)
                        st, en = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                        st.record()
                        f()
                        en.record()
                        torch.cuda.synchronize()
                        coldw[k].append(st.elapsed_time(en))
                cl, cg, cb = (sorted(coldw[k])[5] for k in ("lin", "gem", "bf"))
                rec["cold_write_us"] = {"linear": round(cl * 1e3, 2), "gemm": round(cg * 1e3, 2),
                                        "bf16_linear": round(cb * 1e3, 2)}
                rec["cold_write_gemm_hbm_GB_s"] = round(gb / cg / 1e6, 1)
                del scrub, wscrub
            print(json.dumps(rec), flush=True)
            del xd, wd, bd, wq, sw, xq, sx, y, ws, gws


def recipe(args):
    """The recipe's extra steps: GELU and the SmoothQuant multiplier inside the per-token
    quantizer (against a separate GELU pass), the whole GELU down-projection, the
    multiplier's cost in a linear, and one quantization shared by two linears. One JSON
    line per measurement; times are HIP-graph replays of 20 calls."""
    import numpy as np
    import torch
    import torch.nn.functional as F
    import paper_2606_14598_amd as w8a8
    import synth_inputs as si
    dev = torch.device("cuda:0")

    def emit(rec):
        print(json.dumps(rec), flush=True)

    # 1. quantizer variants on activation matrices of the MLP shapes
    for (M, K, tag) in [(2560, 4096, "attn_in"), (2560, 16384, "mlp_down_in"),
                        (4608, 12288, "paper_ffn_down_in")]:
        h, _, _ = si.make_inputs((M, K, 1), seed=20260 + K, dist="preact")
        hd = dev_bf16(h, dev)
        cm = torch.rand(K, device=dev) * 4 + 0.25
        g = F.gelu(hd)
        base = 3 * M * K + 4 * M
        t = {
            "plain": graph_ms(lambda: w8a8.quantize_act(hd)),
            "colmul": graph_ms(lambda: w8a8.quantize_act(hd, col_mul=cm)),
            "gelu": graph_ms(lambda: w8a8.quantize_act(hd, act="gelu")),
            "gelu_colmul": graph_ms(lambda: w8a8.quantize_act(hd, act="gelu", col_mul=cm)),
            "torch_gelu_then_plain": graph_ms(lambda: w8a8.quantize_act(F.gelu(hd))),
            "torch_gelu_alone": graph_ms(lambda: F.gelu(hd)),
        }
        rec = {"what": "quantizer", "shape": tag, "M": M, "K": K,
               "us": {k: round(v * 1e3, 2) for k, v in t.items()},
               "GB_s": {k: round((base + (4 * K if "colmul" in k else 0)) / t[k] / 1e6, 1)
                        for k in ("plain", "colmul", "gelu", "gelu_colmul")},
               "gelu_fused_speedup_vs_separate_pass": round(t["torch_gelu_then_plain"] / t["gelu"], 3)}
        emit(rec)
        del hd, g, cm

    # 2. the GELU down-projection as one call against GELU + linear and bf16
    for (cfg, name) in [(2, "mlp_down"), (3, "mlp_down")]:
        shp = si.workload(cfg, name)
        M, N, K = shp.M, shp.N, shp.K
        h, w, b = si.make_inputs(shp, dist="preact")
        hd, wd, bd = dev_bf16(h, dev), dev_bf16(w, dev), dev_bf16(b, dev)
        wq, sw = w8a8.quantize_weight(wd)
        y = torch.empty((M, N), dtype=torch.bfloat16, device=dev)
        ws = torch.empty(w8a8.linear_workspace_bytes(M, N, K), dtype=torch.uint8, device=dev)
        fused = graph_ms(lambda: w8a8.linear(hd, wq, sw, bd, act="gelu", out=y, workspace=ws))
        sep = graph_ms(lambda: w8a8.linear(F.gelu(hd), wq, sw, bd, out=y, workspace=ws))
        bf = graph_ms(lambda: F.linear(F.gelu(hd), wd, bd))
        emit({"what": "gelu_down_projection", "config": cfg, "M": M, "K": K, "N": N,
              "us": {"w8a8_linear_gelu": round(fused * 1e3, 2),
                     "torch_gelu_then_w8a8_linear": round(sep * 1e3, 2),
                     "torch_gelu_then_bf16_linear": round(bf * 1e3, 2)},
              "tops_fused": round(gemm_ops(M, N, K) / fused / 1e9, 1),
              "speedup_vs_separate_gelu": round(sep / fused, 3),
              "speedup_vs_bf16": round(bf / fused, 3)})
        del hd, wd, bd, wq, sw, y, ws

    # 3. a smoothed linear (multiplier in the quantizer) against the plain one
    shp = si.workload(1, "attn_proj")
    M, N, K = shp.M, shp.N, shp.K
    x, w, b = si.make_inputs(shp)
    xd, wd, bd = dev_bf16(x, dev), dev_bf16(w, dev), dev_bf16(b, dev)
    ax = w8a8.col_absmax(xd)
    aw = w8a8.col_absmax(wd)
    sm, sm_inv = w8a8.smooth_factors(ax, aw, 0.5)
    wq, sw = w8a8.quantize_weight(wd)
    wqs, sws = w8a8.quantize_weight(wd, col_mul=sm)
    y = torch.empty((M, N), dtype=torch.bfloat16, device=dev)
    ws = torch.empty(w8a8.linear_workspace_bytes(M, N, K), dtype=torch.uint8, device=dev)
    plain = graph_ms(lambda: w8a8.linear(xd, wq, sw, bd, out=y, workspace=ws))
    smooth = graph_ms(lambda: w8a8.linear(xd, wqs, sws, bd, col_mul=sm_inv, out=y, workspace=ws))
    calib = graph_ms(lambda: w8a8.col_absmax(xd, out=ax, accumulate=True))
    emit({"what": "smoothquant_linear", "M": M, "K": K, "N": N,
          "us": {"plain": round(plain * 1e3, 2), "smoothed": round(smooth * 1e3, 2),
                 "calibration_col_absmax_per_batch": round(calib * 1e3, 2)},
          "overhead_pct": round(100 * (smooth / plain - 1), 2)})
    del xd, wd, bd, wq, sw, wqs, sws, y, ws

    # 4. one quantization shared by two linears reading the same activations
    x, _, _ = si.make_inputs((2560, 4096, 1), seed=20261)
    xd = dev_bf16(x, dev)
    lins = []
    for N, seed in ((12288, 11), (16384, 12)):
        _, w, b = si.make_inputs((1, 4096, N), seed=seed)
        wq, sw = w8a8.quantize_weight(dev_bf16(w, dev))
        lins.append((wq, sw, dev_bf16(b, dev), torch.empty((2560, N), dtype=torch.bfloat16,
                                                           device=dev)))
    ws = torch.empty(w8a8.linear_workspace_bytes(2560, 16384, 4096), dtype=torch.uint8,
                     device=dev)
    xq = torch.empty((2560, 4096), dtype=torch.int8, device=dev)

    def two_linears():
        for wq, sw, bd, y in lins:
            w8a8.linear(xd, wq, sw, bd, out=y, workspace=ws)

    def shared():
        q, s = w8a8.quantize_act(xd)
        for wq, sw, bd, y in lins:
            w8a8.gemm(q, s, wq, sw, bd, out=y)

    t2, ts = graph_ms(two_linears), graph_ms(shared)
    emit({"what": "shared_quantization", "M": 2560, "K": 4096, "N": [12288, 16384],
          "us": {"two_linears": round(t2 * 1e3, 2), "quantize_once_two_gemms": round(ts * 1e3, 2)},
          "saving_pct": round(100 * (1 - ts / t2), 2)})


def paper_shapes(args):
    """The paper's five model shapes over its token counts (Section 3, "Target
    architecture"; Section 5 and Table 1): the fused GEMM as it ships (the default plan),
    with the tuned table's tile, with the fallback rule's tile and with one fixed tile
    (the tuning ablation of Section 3, "Why autotuning is load-bearing"), the whole linear
    (per-token quantizer + fused GEMM) and bf16 F.linear, on the same synthetic inputs.
    One JSON line per (shape, M), then one per shape with the ranges over M."""
    import torch
    import torch.nn.functional as F
    import paper_2606_14598_amd as w8a8
    import synth_inputs as si
    dev = torch.device("cuda:0")
    for name, N, K in si.PAPER_SHAPES:
        recs = []
        for M in si.PAPER_M:
            shp = si.paper_shape(name, M)
            x, w, b = si.make_inputs(shp)
            xd = dev_bf16(x, dev)
            del x
            wd, bd = dev_bf16(w, dev), dev_bf16(b, dev)
            wq, sw = w8a8.quantize_weight(wd)
            xq, sx = w8a8.quantize_act(xd)
            y = torch.empty((M, N), dtype=torch.bfloat16, device=dev)
            ws = torch.empty(w8a8.linear_workspace_bytes(M, N, K), dtype=torch.uint8,
                             device=dev)
            ops = gemm_ops(M, N, K)
            it = 20 if ops < 5e14 else 5
            ids = {"tuned": w8a8.select_tile(M, N, K), "default": w8a8.default_tile(M, N, K),
                   "fixed": FIXED_TILE, "plan": -1}
            names = {a: w8a8.plan_name(M, N, K) if i < 0 else w8a8.tile_name(i)
                     for a, i in ids.items()}
            gws = torch.empty(max(1, *(w8a8.gemm_workspace_bytes(M, N, K, i)
                                       for i in ids.values())), dtype=torch.uint8, device=dev)
            t = {}
            for arm, tid in ids.items():
                same = [a for a in t if names[a] == names[arm]]
                t[arm] = t[same[0]] if same else graph_ms(
                    lambda: w8a8.gemm(xq, sx, wq, sw, bd, tile=tid, out=y, workspace=gws), it)
            t["linear"] = graph_ms(lambda: w8a8.linear(xd, wq, sw, bd, out=y, workspace=ws), it)
            t["bf16"] = graph_ms(lambda: F.linear(xd, wd, bd), it)
            rec = {"what": "paper_shape", "shape": name, "M": M, "N": N, "K": K,
                   "tiles": names,
                   "us": {a: round(v * 1e3, 2) for a, v in t.items()},
                   "tops": {a: round(ops / t[a] / 1e9, 1) for a in ("plan", "linear", "bf16")},
                   "gemm_pct_int8_peak": round(100 * ops / t["plan"] / 1e9 / PEAK_INT8_TOPS, 2),
                   "speedup_vs_bf16": {"gemm": round(t["bf16"] / t["plan"], 3),
                                       "gemm_tuned": round(t["bf16"] / t["tuned"], 3),
                                       "gemm_default": round(t["bf16"] / t["default"], 3),
                                       "gemm_fixed": round(t["bf16"] / t["fixed"], 3),
                                       "linear": round(t["bf16"] / t["linear"], 3)},
                   "plan_over_tuned": round(t["tuned"] / t["plan"], 3),
                   "plan_over_default": round(t["default"] / t["plan"], 3),
                   "plan_over_fixed": round(t["fixed"] / t["plan"], 3)}
            print(json.dumps(rec), flush=True)
            recs.append(rec)
            del xd, wd, bd, wq, sw, xq, sx, y, ws, gws
            torch.cuda.empty_cache()

        def rng(key, sub):
            v = [r[key][sub] for r in recs]
            return [min(v), max(v)]
        print(json.dumps({"what": "paper_shape_summary", "shape": name, "N": N, "K": K,
                          "M": si.PAPER_M,
                          "gemm_vs_bf16": rng("speedup_vs_bf16", "gemm"),
                          "gemm_tuned_vs_bf16": rng("speedup_vs_bf16", "gemm_tuned"),
                          "gemm_default_vs_bf16": rng("speedup_vs_bf16", "gemm_default"),
                          "gemm_fixed_vs_bf16": rng("speedup_vs_bf16", "gemm_fixed"),
                          "linear_vs_bf16": rng("speedup_vs_bf16", "linear"),
                          "gemm_tops": rng("tops", "plan")}), flush=True)


def gemm_study(args):
    """The four DiT-block GEMMs at M = 4608 (the headline's dominant kernels), HIP-graph
    replays: the fused GEMM on the workload's codes, on all-zero codes, on constant codes
    and on uniform random codes in [-127, 127] (the same launch, only the operand bits
    change, so the difference is what the matrix cores' switching costs); hipBLASLt's
    int8 GEMM (torch._int_mm, int32 out, no epilogue) and bf16 F.linear on the same
    shapes. One JSON line per shape."""
    import torch
    import torch.nn.functional as F
    import paper_2606_14598_amd as w8a8
    import synth_inputs as si
    dev = torch.device("cuda:0")
    for name in HEADLINE_NAMES:
        shp = si.workload(HEADLINE_CONFIG, name)
        M, N, K = shp.M, shp.N, shp.K
        x, w, b = si.make_inputs(shp)
        xd, wd, bd = dev_bf16(x, dev), dev_bf16(w, dev), dev_bf16(b, dev)
        wq, sw = w8a8.quantize_weight(wd)
        xq, sx = w8a8.quantize_act(xd)
        y = torch.empty((M, N), dtype=torch.bfloat16, device=dev)
        g = torch.Generator(device=dev).manual_seed(shp.seed)
        codes = {
            "workload": (xq, wq),
            "zeros": (torch.zeros_like(xq), torch.zeros_like(wq)),
            "ones": (torch.ones_like(xq), torch.ones_like(wq)),
            "uniform_random": (
                torch.randint(-127, 128, xq.shape, device=dev, dtype=torch.int8, generator=g),
                torch.randint(-127, 128, wq.shape, device=dev, dtype=torch.int8, generator=g)),
        }
        ops = gemm_ops(M, N, K)
        rec = {"what": "gemm_study", "shape": name, "M": M, "K": K, "N": N,
               "tile": w8a8.plan_name(M, N, K),
               "mean_abs_code": {"x": round(float(xq.float().abs().mean()), 2),
                                 "w": round(float(wq.float().abs().mean()), 2)}}
        us, tops = {}, {}
        for k, (a, bq) in codes.items():
            t = graph_ms(lambda: w8a8.gemm(a, sx, bq, sw, bd, out=y), iters=10, warm_ms=40.0)
            us[k], tops[k] = round(t * 1e3, 2), round(ops / t / 1e9, 1)
        wt = wq.t()
        try:
            torch._int_mm(xq, wt)
            t = graph_ms(lambda: torch._int_mm(xq, wt), iters=10, warm_ms=40.0)
            us["hipblaslt_int8_int32_out"], tops["hipblaslt_int8_int32_out"] = (
                round(t * 1e3, 2), round(ops / t / 1e9, 1))
        except Exception as e:  # noqa: BLE001
            rec["hipblaslt_int8"] = f"unavailable: {type(e).__name__}"
        t = graph_ms(lambda: F.linear(xd, wd, bd), iters=10, warm_ms=40.0)
        us["bf16_linear"], tops["bf16_linear"] = round(t * 1e3, 2), round(ops / t / 1e9, 1)
        rec["us"], rec["tops"] = us, tops
        rec["frac_of_peak"] = {k: round(v / PEAK_INT8_TOPS, 4) for k, v in tops.items()}
        print(json.dumps(rec), flush=True)
        del xd, wd, bd, wq, sw, xq, sx, y, codes
        torch.cuda.empty_cache()


def copy_calibration():
    """A plain device copy of known size (for scaling rocprofv3 FETCH_SIZE/WRITE_SIZE)."""
    import torch
    n = 1 << 30
    src = torch.empty(n, dtype=torch.uint8, device="cuda")
    dst = torch.empty(n, dtype=torch.uint8, device="cuda")
    src.fill_(1)
    torch.cuda.synchronize()
    for _ in range(3):
        dst.copy_(src)
    torch.cuda.synchronize()
    print(json.dumps({"copy_bytes_each_way": n, "launches": 3}), flush=True)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=100)
    ap.add_argument("--warmup", type=int, default=100,
                    help="untimed steps first: the chip's power management settles only "
                         "after ~15-20 ms of sustained int8 MFMA load")
    ap.add_argument("--no-cpu", action="store_true", help="skip the CPU-oracle baseline")
    ap.add_argument("--no-extra", action="store_true",
                    help="only the timed step (health gate, comparators, variant skipped)")
    ap.add_argument("--copy-calibration", action="store_true")
    ap.add_argument("--all-shapes", action="store_true",
                    help="time every workload shape (one JSON line each)")
    ap.add_argument("--paper-shapes", action="store_true",
                    help="the paper's five model shapes over M = 512..16384, as shipped and untuned")
    ap.add_argument("--gemm-study", action="store_true",
                    help="the headline GEMMs on workload / zero / constant / random codes, "
                         "beside hipBLASLt int8 and bf16")
    ap.add_argument("--recipe", action="store_true",
                    help="time GELU / SmoothQuant in the quantizer and shared quantization")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py measures one GPU only; --gpus {args.gpus} is not supported "
              "(the path shards by tokens or channels with no exchange between GPUs)",
              file=sys.stderr)
        sys.exit(2)
    if os.environ.get("WORLD_SIZE", "1") not in ("", "1"):
        print("bench.py runs as a single process on one GPU", file=sys.stderr)
        sys.exit(2)
    if args.copy_calibration:
        copy_calibration()
        return
    if args.all_shapes:
        all_shapes(args)
        return
    if args.recipe:
        recipe(args)
        return
    if args.gemm_study:
        gemm_study(args)
        return
    if args.paper_shapes:
        paper_shapes(args)
        return
    rec = run(args)
    print(json.dumps(rec), flush=True)


if __name__ == "__main__":
    main()
