"""Every entry of the GELU quantizer's table against 64 bits (needs an MI355X).

A row that holds one value x alone has the scale |GELU(x)| / 127. The float32 steps of
the table path are the table entry, 1 - h for x >= 0, the product with x and the division
by 127, each rounded once (2^-24): within 2^-22 of the 64-bit value wherever that is a
normal float32."""
import math

import numpy as np
import pytest
import torch

import paper_2606_14598_amd as w8a8

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [8, 2048])
def test_gelu_scale_of_every_magnitude(K):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    # bf16 magnitudes from 2^-30 (below the table's first, 2^-8) to 32 (past its last, 16)
    mag = np.arange((127 - 30) << 7, (127 + 5) << 7, dtype=np.uint16)
    bits = np.concatenate([mag, mag | 0x8000])
    x = torch.from_numpy(bits.view(np.int16)).view(torch.bfloat16).cuda()
    rows = x[:, None].expand(-1, K).contiguous()
    q, s = w8a8.quantize_act(rows, act="gelu")
    v = x.double().cpu().numpy()
    want = np.abs([0.5 * t * math.erfc(-t / math.sqrt(2.0)) for t in v]) / 127.0
    got = s.double().cpu().numpy()
    normal = want > 2.0 ** -120
    assert normal.sum() > 0.8 * want.size
    rel = np.abs(got[normal] - want[normal]) / want[normal]
    print(f"K={K}: worst relative scale error {rel.max():.3g}", flush=True)
    assert rel.max() <= 2.0 ** -22
    sign = np.where(v > 0, 127, -127)[normal]
    assert (q.cpu().numpy()[normal] == sign[:, None]).all()
