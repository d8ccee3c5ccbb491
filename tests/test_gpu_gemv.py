"""Up to 8 tokens: the row-reading kernel of w8a8.linear and w8a8.gemm against the oracle's codes
and product and, bit for bit, against a streaming tile (needs an MI355X). K at the edges of a
16-byte chunk, a kilobyte and a turn of each variant; channel counts around a wavefront's and
a workgroup's rows."""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_14598_amd as w8a8
import synth_inputs as si
from _helpers import dev_bf16, host_bits, say, ulp_distance

pytestmark = pytest.mark.gpu

TILE = "wsx_m16n16w8d4"


@pytest.mark.parametrize("K", [16, 1008, 1024, 1040, 2032, 2048, 2064, 4080, 4096, 4112, 8176,
                               8192, 8208, 16368, 16384, 16400])
def test_one_token(K):
    tile = [w8a8.tile_name(i) for i in range(w8a8.tile_count())].index(TILE)
    for N in (1, 3, 4, 7, 8, 9, 15, 17, 33, 300):
        say(f"one token K={K} N={N}")
        x, w, b = si.make_inputs((1, K, N), seed=K + N, dist="outlier")
        wq_o, sw_o = oracle.quantize_rows(w)
        y_o = oracle.linear(x, wq_o, sw_o, b)[0]
        xd, bd = dev_bf16(x), dev_bf16(b)
        wq, sw = w8a8.quantize_weight(dev_bf16(w))
        xq, sx = w8a8.quantize_act(xd)
        want = host_bits(w8a8.gemm(xq, sx, wq, sw, bd, tile=tile))
        assert ulp_distance(want, y_o).max() <= 1
        assert np.array_equal(host_bits(w8a8.gemm(xq, sx, wq, sw, bd)), want)
        assert np.array_equal(host_bits(w8a8.linear(xd, wq, sw, bd)), want)
        assert np.array_equal(host_bits(w8a8.gemm(xq, sx, wq, sw)),
                              host_bits(w8a8.gemm(xq, sx, wq, sw, tile=tile)))
        # the guard behind the last output stays
        buf = torch.full((N + 8,), 5.0, dtype=torch.bfloat16, device="cuda")
        w8a8.linear(xd, wq, sw, bd, out=buf[:N].view(1, N))
        assert np.array_equal(host_bits(buf[:N].view(1, N)), want) and (buf[N:] == 5.0).all()


@pytest.mark.parametrize("K", [16, 1040, 2048, 2064, 4096, 4112, 8192, 16384, 16400, 32768])
def test_few_tokens(K):
    tile = [w8a8.tile_name(i) for i in range(w8a8.tile_count())].index("m32n128k128w1x4s6")
    # five tokens and more take the kernel only on 16384 channels with a weight of 32 MB
    wide = [(5, 16400), (8, 8193), (8, 16387)] if K == 4096 else [(7, 16385)] if K == 2048 else []
    for M, N in [(m, n) for m in (2, 3, 4) for n in (1, 3, 8, 17, 130)] + wide:
        say(f"few tokens M={M} K={K} N={N}")
        x, w, b = si.make_inputs((M, K, N), seed=M + K + N, dist="outlier")
        wq, sw = w8a8.quantize_weight(dev_bf16(w))
        xq, sx = w8a8.quantize_act(dev_bf16(x))
        bd = dev_bf16(b)
        want = host_bits(w8a8.gemm(xq, sx, wq, sw, bd, tile=tile))
        out = torch.full((M * N + 8,), 5.0, dtype=torch.bfloat16, device="cuda")
        y = w8a8.gemm(xq, sx, wq, sw, bd, out=out[:M * N].view(M, N))
        assert np.array_equal(host_bits(y), want) and (out[M * N:] == 5.0).all()
        assert np.array_equal(host_bits(w8a8.linear(dev_bf16(x), wq, sw, bd)), want)


def test_one_token_zero_row():
    wq, sw = w8a8.quantize_weight(torch.randn(40, 4096, device="cuda").bfloat16())
    bias = torch.randn(40, device="cuda").bfloat16()
    y = w8a8.linear(torch.zeros(1, 4096, device="cuda", dtype=torch.bfloat16), wq, sw, bias)
    assert torch.equal(y[0], bias)
