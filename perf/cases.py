"""Performance cases of the fused W8A8 linear: what a diffusion transformer's inference
program has this library do, from one conditioning token to a whole block at 1024px.

A case is a dict of plain values. Its "kind" is the way the program calls the library:

  linear     w8a8.linear on one activation matrix (quantizer + GEMM + epilogue)
  module     the W8A8Linear drop-in module (the torch.library op) on one matrix
  graph      `layers` linears, each with its own weights, captured once in a HIP graph
             with caller-provided outputs and workspace; a pass is one replay
  shared     quantize_act once, then w8a8.gemm for each linear that reads the same
             activations
  block      the four linears of a transformer block as W8A8Linear modules (the MLP's
             down-projection consumes the pre-activation of its GELU)
  calibrate  preparing one layer: column maxima of activations and weights, SmoothQuant
             factors, weight quantization

M tokens, K input channels, N output channels; "act" is the transform in front of the
quantizer, "smooth" the SmoothQuant multiplier, "bias" a bf16 bias. Sizes are those of
the 4096-wide DiT family (768px: 2560 tokens, 1024px: 4608), of the 4608-wide model and
its LLM projection, and of the few-token and odd shapes around them.
"""
import math

import torch

import paper_2606_14598_amd as w8a8
from paper_2606_14598_amd.torch_ops import W8A8Linear

# Largest work of a drawn case, in int8 ops (the listed block has 1.63e12).
MAX_OPS = 8e11


def _case(name, kind, M, K, N, act="none", smooth=False, bias=True, **more):
    return dict(name=name, kind=kind, M=M, K=K, N=N, act=act, smooth=smooth, bias=bias, **more)


def listed():
    return [
        # The smallest call: a small projection of a short sequence, bound by latency.
        _case("tiny", "linear", 64, 256, 128),
        # Text conditioning through the drop-in module, as eager code calls it.
        _case("text_module", "module", 77, 4096, 16384),
        # One conditioning vector (timestep embedding) through the modulation linears of
        # four blocks, captured in a graph as a launch-bound sampler does.
        _case("one_token_graph", "graph", 1, 4096, 16384, layers=4),
        # A few hundred tokens (text plus a thumbnail) with SmoothQuant, captured.
        _case("few_hundred_graph", "graph", 333, 4096, 4096, smooth=True, layers=4),
        # 768px attention projection.
        _case("attn_768", "linear", 2560, 4096, 4096),
        # 1024px MLP up-projection with SmoothQuant.
        _case("mlp_up_1024", "linear", 4608, 4096, 16384, smooth=True),
        # 1024px MLP down-projection, GELU and SmoothQuant folded into its quantizer.
        _case("mlp_down_1024", "linear", 4608, 16384, 4096, act="gelu", smooth=True),
        # Odd sizes: channels that are no multiple of a vector load, ragged tokens, no bias.
        _case("ragged", "linear", 2001, 1000, 3001, bias=False),
        # The LLM projection: a very long K at few tokens.
        _case("llm_proj", "linear", 512, 53248, 4608),
        # qkv and MLP up-projection of a parallel block reading one quantized activation.
        _case("shared_768", "shared", 2560, 4096, 12288, N2=16384),
        # Preparing the MLP up-projection: calibration and weight quantization.
        _case("calibrate_layer", "calibrate", 4608, 4096, 16384, smooth=True, bias=False),
        # The largest: a 4608-wide block at its 1024px token count.
        _case("block_4608", "block", 4110, 4608, 12288, smooth=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges: sizes log-uniform, a quarter of them with
    channel counts of any residue, the others multiples of 16 (as model widths are)."""
    kind = rng.choice(["linear", "linear", "linear", "module", "graph", "shared",
                       "calibrate", "block"])
    ragged = rng.random() < 0.25
    unit = 1 if ragged else 16
    act = rng.choice(["none", "none", "gelu"])
    smooth = rng.random() < 0.5
    bias = rng.random() < 0.75
    cap, k_max = (4e10, 8192) if ragged else (MAX_OPS, 24576)
    while True:
        M = _log(rng, 1, 384) if kind in ("module", "graph") else _log(rng, 1, 8192)
        K = max(unit, _log(rng, 256, k_max) // unit * unit)
        N = max(unit, _log(rng, 128, 20480) // unit * unit)
        if kind == "calibrate":
            # calibration batches are long, layers whole
            M, smooth, act, bias = max(M, 256), True, "none", False
        if kind == "block":
            M = max(M, 128)
            K = max(256, min(K, 5120))
            N = 4 * K
            if 2.0 * M * K * 4 * K + 4.0 * M * K * N > cap:
                continue
            return _strip(_case("", kind, M, K, N, smooth=smooth, bias=bias))
        if kind == "shared":
            N2 = max(unit, _log(rng, 128, 20480) // unit * unit)
            if 2.0 * M * K * (N + N2) > cap:
                continue
            return _strip(_case("", kind, M, K, N, act, smooth, bias, N2=N2))
        if kind == "graph":
            return _strip(_case("", kind, M, K, N, act, smooth, bias,
                                layers=rng.randint(1, 4)))
        if 2.0 * M * K * N <= cap:
            return _strip(_case("", kind, M, K, N, act, smooth, bias))


def _strip(case):
    del case["name"]
    return case


# ---------------------------------------------------------------- inputs

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _x(g, M, K, act):
    """Activations: N(0, 1), two outlier channels x20 unless they are the pre-activation
    of a GELU."""
    x = torch.randn((M, K), generator=g, device="cuda", dtype=torch.float32)
    if act == "none":
        for c in sorted({17, 3 * K // 4 + 5}):
            if c < K:
                x[:, c] *= 20.0
    return x.to(torch.bfloat16)


def _w(g, N, K):
    """Weights: N(0, 0.02) times a per-output-channel factor from U(0.5, 2)."""
    w = torch.randn((N, K), generator=g, device="cuda", dtype=torch.float32)
    w *= 0.02 * (0.5 + 1.5 * torch.rand((N, 1), generator=g, device="cuda"))
    return w.to(torch.bfloat16)


def _b(g, N, bias):
    if not bias:
        return None
    return (0.01 * torch.randn(N, generator=g, device="cuda")).to(torch.bfloat16)


def _layer(g, x, N, act, smooth, bias):
    """(wq, sw, b, s_inv) of one calibrated and quantized linear that reads x."""
    w = _w(g, N, x.shape[1])
    s = si = None
    if smooth:
        s, si = w8a8.smooth_factors(w8a8.col_absmax(x, act=act), w8a8.col_absmax(w))
    wq, sw = w8a8.quantize_weight(w, col_mul=s)
    return wq, sw, _b(g, N, bias), si


def _block_parts(case):
    """(input, N, act) of the block's linears: qkv, attention out, MLP up, MLP down."""
    K, N = case["K"], case["N"]
    return [("x", 3 * K, "none"), ("a", K, "none"), ("h", N, "none"), (None, K, "gelu")]


def prepare(case, seed):
    g = _gen(seed)
    kind, M, K, N = case["kind"], case["M"], case["K"], case["N"]
    act, smooth, bias = case["act"], case["smooth"], case["bias"]
    st = {"kind": kind, "act": act}
    if kind == "calibrate":
        st["x"], st["w"] = _x(g, M, K, act), _w(g, N, K)
        return st
    if kind == "block":
        for n in ("x", "a", "h"):
            st[n] = _x(g, M, K, "none")
        mods = []
        for src, n, a in _block_parts(case):
            x = st[src] if src else _x(g, min(M, 512), N, "gelu")
            wq, sw, b, si = _layer(g, x, n, a, smooth, bias)
            mods.append(W8A8Linear(wq, sw, b, act=a, smooth_inv=si))
        st["mods"] = mods
        return st
    x = st["x"] = _x(g, M, K, act)
    if kind == "graph":
        st["layers"] = [_layer(g, x, N, act, smooth, bias) for _ in range(case["layers"])]
        st["out"] = [torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
                     for _ in st["layers"]]
        ws = st["ws"] = torch.empty(w8a8.linear_workspace_bytes(M, N, K), dtype=torch.uint8,
                                    device="cuda")

        def calls():
            for (wq, sw, b, si), y in zip(st["layers"], st["out"]):
                w8a8.linear(x, wq, sw, b, act=act, col_mul=si, out=y, workspace=ws)
        calls()
        graph = st["graph"] = torch.cuda.CUDAGraph()
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            with torch.cuda.graph(graph, stream=s):
                calls()
        torch.cuda.current_stream().wait_stream(s)
        return st
    st["w"] = [_layer(g, x, N, act, smooth, bias)]
    if kind == "shared":
        # one smoothing serves both linears: the second weight takes the first's factors
        wq, sw, b, si = st["w"][0]
        s = None if si is None else 1.0 / si
        wq2, sw2 = w8a8.quantize_weight(_w(g, case["N2"], K), col_mul=s)
        st["w"].append((wq2, sw2, _b(g, case["N2"], bias), si))
    if kind == "module":
        wq, sw, b, si = st["w"][0]
        st["mod"] = W8A8Linear(wq, sw, b, act=act, smooth_inv=si)
    return st


def run(st):
    kind = st["kind"]
    if kind == "linear":
        wq, sw, b, si = st["w"][0]
        return w8a8.linear(st["x"], wq, sw, b, act=st["act"], col_mul=si)
    if kind == "module":
        with torch.no_grad():
            return st["mod"](st["x"])
    if kind == "graph":
        st["graph"].replay()
        return st["out"]
    if kind == "shared":
        xq, sx = w8a8.quantize_act(st["x"], act=st["act"], col_mul=st["w"][0][3])
        return [xq, sx] + [w8a8.gemm(xq, sx, wq, sw, b) for wq, sw, b, _ in st["w"]]
    if kind == "block":
        qkv, out, up, down = st["mods"]
        with torch.no_grad():
            h = up(st["h"])
            return [qkv(st["x"]), out(st["a"]), h, down(h)]
    ax = w8a8.col_absmax(st["x"])
    aw = w8a8.col_absmax(st["w"])
    s, si = w8a8.smooth_factors(ax, aw)
    wq, sw = w8a8.quantize_weight(st["w"], col_mul=s)
    return [ax, aw, s, si, wq, sw]


# ---------------------------------------------------------------- accounting

def _linear_bytes(M, K, N, smooth, bias):
    return 2 * M * K + N * K + 2 * M * N + 4 * N + (4 * K if smooth else 0) + \
        (2 * N if bias else 0)


def work(case):
    """X, the weight codes, scales, bias and multiplier read once, Y written once; 2 ops
    per multiply-accumulate. Quantized activations count only where they are an output."""
    kind, M, K, N = case["kind"], case["M"], case["K"], case["N"]
    sm, bi = case["smooth"], case["bias"]
    if kind == "calibrate":
        return {"bytes": 2 * M * K + 2 * N * K + N * K + 4 * N + 16 * K, "flops": 4.0 * N * K}
    if kind == "block":
        parts = [(K, 3 * K), (K, K), (K, N), (N, K)]
        return {"bytes": sum(_linear_bytes(M, k, n, sm, bi) for k, n in parts),
                "flops": sum(2.0 * M * k * n for k, n in parts)}
    if kind == "shared":
        n2 = case["N2"]
        return {"bytes": 3 * M * K + 4 * M + (N + n2) * (K + 4 + 2 * M)
                + (4 * K if sm else 0) + (2 * (N + n2) if bi else 0),
                "flops": 2.0 * M * K * (N + n2)}
    layers = case.get("layers", 1)
    return {"bytes": layers * _linear_bytes(M, K, N, sm, bi) - (layers - 1) * 2 * M * K,
            "flops": layers * 2.0 * M * K * N}


def tolerance(case):
    """bf16 results of an exact integer product: the rounding of the output (2^-9, 1.7e-3
    in the 2-norm against 64 bits) and codes that fall the other way at a rounding tie.
    Calibration: float32 maxima are exact, the factors a few float32 roundings."""
    if case["kind"] == "calibrate":
        return {"rel": 1e-6, "max": 1e-5, "differ": 1e-5}
    return {"rel": 7e-3, "max": 0.05, "differ": 1e-4}


# ---------------------------------------------------------------- 64-bit results

def _transform(x, act, si):
    v = x.double()
    if act == "gelu":
        v = 0.5 * v * torch.erfc(v * -math.sqrt(0.5))
    return v if si is None else v * si.double()


def _quantize(v):
    a = v.abs().amax(dim=1)
    inv = torch.where(a > 0, 127.0 / a, torch.zeros_like(a))
    return torch.round(v * inv[:, None]).clamp_(-127, 127), a / 127.0


def _product(q, sx, wq, sw, b):
    y = torch.matmul(q, wq.double().t()) * (sx[:, None] * sw.double()[None, :])
    return y if b is None else y + b.double()


def exact(case, seed):
    st = prepare(case, seed)
    kind, act = st["kind"], st["act"]
    if kind == "calibrate":
        ax, aw = st["x"].double().abs().amax(0), st["w"].double().abs().amax(0)
        ok = (ax > 0) & (aw > 0)
        s = torch.where(ok, torch.sqrt(ax) / torch.sqrt(aw), torch.ones_like(ax))
        q, sw = _quantize(st["w"].double() * s)
        return [ax, aw, s, 1.0 / s, q.to(torch.int8), sw]
    if kind == "block":
        outs, h = [], None
        for (src, _, a), m in zip(_block_parts(case), st["mods"]):
            # the module's own input is the bf16 tensor the up-projection hands on
            x = st[src] if src else h.to(torch.bfloat16)
            q, sx = _quantize(_transform(x, a, m.smooth_inv))
            y = _product(q, sx, m.wq, m.w_scale, m.bias)
            h = y
            outs.append(y)
        return outs
    if kind == "graph":
        q = [_quantize(_transform(st["x"], act, si)) for _, _, _, si in st["layers"]]
        return [_product(*qs, wq, sw, b) for qs, (wq, sw, b, _) in zip(q, st["layers"])]
    q, sx = _quantize(_transform(st["x"], act, st["w"][0][3]))
    ys = [_product(q, sx, wq, sw, b) for wq, sw, b, _ in st["w"]]
    return [q.to(torch.int8), sx] + ys if kind == "shared" else ys[0]
