"""Column maxima against the oracle at the edges of the kernel's mapping (needs an MI355X):
lanes per row (1 to 64), a ragged last vector, K < 8, one block of rows or several, both
block sizes; and the three candidates of |GELU| over every bf16 magnitude."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2606_14598_amd as w8a8
import synth_inputs as si

pytestmark = pytest.mark.gpu


def _dev(bits):
    return torch.from_numpy(bits.view(np.int16)).view(torch.bfloat16).cuda()


@pytest.mark.parametrize("rows,K", [(1, 1), (3, 7), (9, 8), (130, 9), (129, 513), (600, 520),
                                    (2100, 77), (4099, 33), (300, 4100)])
def test_col_absmax_shapes(rows, K):
    x, _, _ = si.make_inputs((rows, K, 1), seed=rows + K)
    out = w8a8.col_absmax(_dev(x))
    assert np.array_equal(out.cpu().numpy(), oracle.col_absmax(x))
    # rows at an odd element offset, merged into larger and smaller values
    buf = torch.empty(rows * K + 1, dtype=torch.bfloat16, device="cuda")
    v = buf[1:].view(rows, K)
    v.copy_(_dev(x))
    have = np.where(np.arange(K) % 2 == 0, 1e-3, 1e3).astype(np.float32)
    out = torch.from_numpy(have).cuda()
    w8a8.col_absmax(v, out=out, accumulate=True)
    assert np.array_equal(out.cpu().numpy(), np.maximum(have, oracle.col_absmax(x)))


def test_col_absmax_gelu_every_magnitude():
    # Column j holds one bf16 value of either sign and one smaller magnitude, so each side
    # of the peak of |x| Phi(-|x|) and each order of the two decides in some column. The
    # bound is that of the erfc fit (a few float32 roundings, see test_gpu_transforms.py).
    mag = np.arange((127 - 20) << 7, (127 + 3) << 7, dtype=np.uint16)
    neg = mag | 0x8000
    x = np.stack([neg, np.roll(neg, 40), np.roll(mag, 900)])
    x[2, ::2] = 0
    got = w8a8.col_absmax(_dev(x), act="gelu").cpu().numpy().astype(np.float64)
    v = oracle.bf16_to_f32(x).astype(np.float64)
    g = np.abs([[0.5 * t * math.erfc(-t / math.sqrt(2.0)) for t in row] for row in v])
    assert np.max(np.abs(got / g.max(axis=0) - 1)) <= 2.0 ** -17


def test_col_absmax_special_values():
    inf, nan = float("inf"), float("nan")
    x = torch.tensor([[1.0, -inf, nan, -3.0, inf, -0.0], [2.0, 5.0, 7.0, -0.5, -1.0, 0.0]],
                     dtype=torch.bfloat16, device="cuda")
    m = w8a8.col_absmax(x).cpu()
    assert m[[0, 1, 3, 4, 5]].tolist() == [2.0, inf, 3.0, inf, 0.0] and math.isnan(m[2])
    g = w8a8.col_absmax(x, act="gelu").cpu()
    # GELU(-inf) is -inf * 0
    assert math.isnan(g[1]) and math.isnan(g[2]) and g[4] == inf and g[5] == 0.0


@pytest.mark.parametrize("K", [3, 8, 64, 70, 256, 520, 1001, 4096])
def test_col_absmax_block_sizes(K):
    """Row counts at the edges of the launch rule: one block of 64 to 1024 threads, several
    of 64 to 1024, and the last partial one."""
    lanes = min(64, 1 << (-(-K // 8) - 1).bit_length())
    one = {8 * max(1, t // lanes) for t in (64, 128, 256, 512, 1024)}
    for rows in sorted({1, *one, *(r + 1 for r in one), 4 * max(one), 4 * max(one) + 1}):
        x, _, _ = si.make_inputs((rows, K, 1), seed=rows + K, dist="preact")
        assert np.array_equal(w8a8.col_absmax(_dev(x)).cpu().numpy(), oracle.col_absmax(x)), rows
        if rows <= 600:
            g = w8a8.col_absmax(_dev(x), act="gelu").cpu().numpy()
            want = oracle.col_absmax(x, act="gelu")
            assert np.all(np.abs(g - want) <= 2.0 ** -17 * want), rows
