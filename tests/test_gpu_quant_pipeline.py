"""The register-resident quantizer's row pipeline against the oracle (needs an MI355X): more
rows than the grid holds (two to four turns, the last one partial) for one wavefront to a
whole block per row, and rows whose 8-byte vectors do not pair up (K % 16 == 8)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_14598_amd as w8a8
import synth_inputs as si
from _gelu_checks import check_gelu_codes
from _helpers import dev_bf16, dev_f32, host, say

pytestmark = pytest.mark.gpu

CASES = [(8193, 8), (24581, 24), (16390, 520), (9001, 1032), (8195, 2056), (4100, 4104),
         (2049, 4616), (4099, 6152), (1500, 9224), (1030, 12296), (770, 16376), (1100, 16384),
         (515, 20488), (1, 16), (3, 40000)]


@pytest.mark.parametrize("rows,K", CASES)
def test_rows_beyond_the_grid(rows, K):
    say(f"quantizer rows={rows} K={K}")
    x, _, _ = si.make_inputs((rows, K, 1), seed=rows + K, dist="outlier")
    x[rows // 2] = 0
    xd = dev_bf16(x)
    q_o, s_o = oracle.quantize_rows(x)
    q, s = w8a8.quantize_act(xd)
    assert np.array_equal(host(q), q_o) and np.array_equal(host(s), s_o)
    cm = np.random.default_rng(K).uniform(0.05, 8, K).astype(np.float32)
    q_o, s_o = oracle.quantize_rows(x, col_mul=cm)
    q, s = w8a8.quantize_act(xd, col_mul=dev_f32(cm))
    assert np.array_equal(host(q), q_o) and np.array_equal(host(s), s_o)


@pytest.mark.parametrize("rows,K", [(8193, 264), (2050, 4104), (300, 2568), (1030, 16376)])
def test_gelu_rows_beyond_the_grid(rows, K):
    say(f"gelu quantizer rows={rows} K={K}")
    x, _, _ = si.make_inputs((rows, K, 1), seed=rows, dist="preact")
    q_o, s_o = oracle.quantize_rows(x, act="gelu")
    q, s = w8a8.quantize_act(dev_bf16(x), act="gelu")
    check_gelu_codes(x, host(q), host(s), q_o, s_o, None, f"{rows}x{K}")


@pytest.mark.parametrize("rows,K", [(3, 16392), (1030, 20488), (515, 24576), (3, 24584)])
def test_three_vectors_a_thread(rows, K):
    """The edges of the 1024 x 3 mapping, with every transform."""
    say(f"quantizer 1024 x 3 rows={rows} K={K}")
    x, _, _ = si.make_inputs((rows, K, 1), seed=rows + K, dist="preact")
    cm = np.random.default_rng(K).uniform(0.05, 8, K).astype(np.float32)
    for act in ("none", "gelu"):
        for c in (None, cm):
            q_o, s_o = oracle.quantize_rows(x, act=act, col_mul=c)
            q, s = w8a8.quantize_act(dev_bf16(x), act=act,
                                     col_mul=None if c is None else dev_f32(c))
            if act == "none":
                assert np.array_equal(host(q), q_o) and np.array_equal(host(s), s_o)
            else:
                check_gelu_codes(x, host(q), host(s), q_o, s_o, c, f"{rows}x{K}")


def test_output_rows_at_eight_bytes():
    """Codes into rows at an 8-byte offset: no 16-byte streaming stores."""
    lib = w8a8.load_library()
    rows, K = 300, 4096
    x, _, _ = si.make_inputs((rows, K, 1), seed=3)
    xd = dev_bf16(x)
    buf = torch.full((rows * K + 24,), 85, dtype=torch.int8, device="cuda")
    s = torch.empty(rows, dtype=torch.float32, device="cuda")
    st = lib.w8a8_quantize_act(xd.data_ptr(), rows, K, buf.data_ptr() + 8, s.data_ptr(),
                               torch.cuda.current_stream().cuda_stream)
    assert st == 0
    q_o, s_o = oracle.quantize_rows(x)
    got = host(buf)
    assert np.array_equal(got[8:8 + rows * K].reshape(rows, K), q_o)
    assert np.array_equal(host(s), s_o) and (got[:8] == 85).all() and (got[8 + rows * K:] == 85).all()
