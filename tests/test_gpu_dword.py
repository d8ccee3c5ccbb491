"""Operands that are only 4-byte aligned (K % 4 == 0 but not % 16, or such pointers) on the
direct-to-LDS tiles: exact accumulators against the oracle for every such tile, at the edges
of a chunk (16 bytes), of a panel and of the ring, with K split and not (needs an MI355X).
Every byte around the operands is nonzero, so a row's end that is not cut off shows."""
import re

import numpy as np
import pytest
import torch

import oracle
import paper_2606_14598_amd as w8a8

pytestmark = pytest.mark.gpu


def _tiles():
    out = []
    for i in range(w8a8.tile_count()):
        m = re.match(r"m(\d+)n(\d+)k(\d+)w\d+x\d+s(\d+)$", w8a8.tile_name(i))
        if m and int(m[4]) >= 3:
            out.append((i, int(m[1]), int(m[2]), int(m[3]), int(m[4])))
    return out


def _at(a, off):
    """The int8 matrix at byte offset off of a buffer of other nonzero bytes."""
    buf = torch.full((a.size + off + 64,), 101, dtype=torch.int8, device="cuda")
    v = buf[off:off + a.size].view(a.shape)
    v.copy_(torch.from_numpy(a))
    return v


def _codes(rng, *shape):
    v = rng.integers(1, 128, shape) * rng.choice([-1, 1], shape)
    return v.astype(np.int8)


@pytest.mark.parametrize("tile,tm,tn,bk,stages", _tiles())
def test_every_dword_tile(tile, tm, tn, bk, stages):
    rng = np.random.default_rng(tile)
    for K in (4, 12, 20, bk - 4, bk, bk + 4, 2 * bk - 12, (stages - 1) * bk + 8, stages * bk + 36):
        for M, N in ((tm + 33, tn - 5), (max(33, tm - 1), tn + 1)):
            print(f"dword tile {w8a8.tile_name(tile)} M={M} N={N} K={K}", flush=True)
            xq, wq = _codes(rng, M, K), _codes(rng, N, K)
            want = oracle.gemm_acc(xq, wq)
            for ox, ow in ((4, 0), (8, 12)):
                got = w8a8.gemm_acc_i32(_at(xq, ox), _at(wq, ow), tile=tile)
                assert np.array_equal(got.cpu().numpy(), want), (M, N, K, ox, ow)


@pytest.mark.parametrize("M,N,K,split", [(33, 640, 24572, True), (146, 1361, 18980, True),
                                         (512, 1152, 13324, True), (2001, 3001, 1000, False),
                                         (64, 64, 4100, True), (4500, 130, 260, False)])
def test_dword_default_plan(M, N, K, split):
    print(f"dword plan M={M} N={N} K={K}", flush=True)
    assert (w8a8.gemm_workspace_bytes(M, N, K) > 0) == split
    rng = np.random.default_rng(K)
    xq, wq = _codes(rng, M, K), _codes(rng, N, K)
    sx = (rng.random(M) + 0.5).astype(np.float32)
    sw = (rng.random(N) + 0.5).astype(np.float32)
    acc = torch.from_numpy(xq).double() @ torch.from_numpy(wq).double().t()   # exact
    scale = torch.from_numpy(sx)[:, None] * torch.from_numpy(sw)[None, :]
    want = (acc.float() * scale).bfloat16()
    y = w8a8.gemm(_at(xq, 4), torch.from_numpy(sx).cuda(), _at(wq, 8),
                  torch.from_numpy(sw).cuda())
    assert torch.equal(y.cpu(), want)
