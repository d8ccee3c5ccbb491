"""The default plan of a GEMM (tile and K split by the cost model) against a fixed unsplit
tile: the int32 sums are exact, so the bits must be equal (needs an MI355X). Shapes where
the plan splits K, is at its limits (17 tokens, a short last K-range, channels that are no
multiple of 4) or falls back for want of workspace."""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_14598_amd as w8a8
import synth_inputs as si
from _helpers import dev_bf16, host_bits, say, ulp_distance

pytestmark = pytest.mark.gpu

PLAIN_TILE = "m128n128k128w2x2s4"

# (M, N, K, whether the default plan needs partials)
SHAPES = [(17, 224, 14208, False), (33, 640, 24576, True), (49, 1216, 18304, True),
          (128, 560, 18192, True), (129, 130, 8208, True), (146, 1361, 18976, True),
          (300, 99, 24576, True), (512, 1152, 13328, True), (1000, 2000, 20000, True),
          (4576, 144, 19184, True), (640, 1024, 4096, False), (17, 16, 16, False),
          (40, 3000, 1040, False), (8192, 129, 272, False)]


def _tile(name):
    return [w8a8.tile_name(i) for i in range(w8a8.tile_count())].index(name)


def _operands(M, N, K, seed):
    x, w, b = si.make_inputs((M, K, N), seed=seed)
    wq, sw = w8a8.quantize_weight(dev_bf16(w))
    xd = dev_bf16(x)
    xq, sx = w8a8.quantize_act(xd)
    return x, w, b, xd, xq, sx, wq, sw, dev_bf16(b)


@pytest.mark.parametrize("M,N,K,split", SHAPES)
def test_default_plan_matches_the_plain_tile(M, N, K, split):
    say(f"plan M={M} N={N} K={K}")
    need = w8a8.gemm_workspace_bytes(M, N, K)
    assert (need > 0) == split
    _, _, _, xd, xq, sx, wq, sw, bd = _operands(M, N, K, M + N)
    want = host_bits(w8a8.gemm(xq, sx, wq, sw, bd, tile=_tile(PLAIN_TILE)))
    assert np.array_equal(host_bits(w8a8.gemm(xq, sx, wq, sw, bd)), want)
    assert np.array_equal(host_bits(w8a8.linear(xd, wq, sw, bd)), want)
    want = host_bits(w8a8.gemm(xq, sx, wq, sw, tile=_tile(PLAIN_TILE)))
    assert np.array_equal(host_bits(w8a8.gemm(xq, sx, wq, sw)), want)
    # a workspace of the least size (and one byte less than the plan's)
    lib = w8a8.load_library()
    least = lib.w8a8_linear_workspace_least_bytes(M, N, K)
    full = w8a8.linear_workspace_bytes(M, N, K)
    assert least <= full and (least < full or not split or M <= 128)
    for n in {least, max(least, full - 1)}:
        y = w8a8.linear(xd, wq, sw, workspace=torch.empty(n, dtype=torch.uint8, device="cuda"))
        assert np.array_equal(host_bits(y), want), n
    with pytest.raises(ValueError):
        w8a8.linear(xd, wq, sw, workspace=torch.empty(least - 1, dtype=torch.uint8,
                                                      device="cuda"))


def test_split_plan_under_graph_replays():
    M, N, K = 300, 1361, 16400
    assert w8a8.gemm_workspace_bytes(M, N, K) > 0
    _, _, _, xd, _, _, wq, sw, bd = _operands(M, N, K, 5)
    want = host_bits(w8a8.linear(xd, wq, sw, bd))
    y = torch.empty(M, N, dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(w8a8.linear_workspace_bytes(M, N, K), dtype=torch.uint8, device="cuda")
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        w8a8.linear(xd, wq, sw, bd, out=y, workspace=ws)
    for _ in range(3):
        y.zero_()
        ws.fill_(0x5A)
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(host_bits(y), want)


def test_split_plan_against_the_oracle():
    M, N, K = 130, 70, 8208
    assert w8a8.gemm_workspace_bytes(M, N, K) > 0
    x, w, b, xd, _, _, wq, sw, bd = _operands(M, N, K, 9)
    wq_o, sw_o = oracle.quantize_rows(w)
    y_o = oracle.linear(x, wq_o, sw_o, b)[0]
    assert ulp_distance(host_bits(w8a8.linear(xd, wq, sw, bd)), y_o).max() <= 1
