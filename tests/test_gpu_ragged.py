"""Operands at any alignment and any K: the kernels behind K % 16 != 0 and unaligned
pointers against the oracle, at the edges of their panels and tiles (needs an MI355X).

Codes, scales and accumulators are exact integers or correctly rounded single steps, so
they must match bit for bit; the bf16 outputs run the oracle's own float32 chain and are
held to the parity bar of the other tests (1 ulp, cosine)."""
import numpy as np
import pytest
import torch

import oracle
import synth_inputs as si
import paper_2606_14598_amd as w8a8
from _helpers import assert_bf16_parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w8a8.load_library()
    yield
    torch.cuda.synchronize()


def dev_bf16(bits):
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).view(torch.bfloat16).cuda()


def host_bits(t):
    return t.contiguous().view(torch.int16).cpu().numpy().view(np.uint16)


def at_offset(t: torch.Tensor, off: int) -> torch.Tensor:
    """The same values in a contiguous view whose first byte is off elements into a
    larger buffer filled with a canary."""
    buf = torch.full((t.numel() + off + 64,), 77, dtype=t.dtype, device=t.device)
    v = buf[off:off + t.numel()].view(t.shape)
    v.copy_(t)
    return v


# One (M, N) per kernel of the any-alignment dispatch: 16 and 32 tokens of the streaming
# kernel, then the 64 x 64, 128 x 64, 128 x 128 and 256 x 256 tiles, each ragged.
ANY_SHAPES = [(1, 33), (16, 130), (17, 65), (32, 49), (33, 77), (130, 500), (600, 2000),
              (2001, 3001), (4090, 4001)]
# K around a 16-byte chunk, a panel (128) and a super-step (256), single bytes included.
ANY_K = [1, 9, 15, 17, 127, 129, 200, 255, 257, 1000, 2049]


@pytest.mark.parametrize("M,N", ANY_SHAPES)
def test_any_alignment_linear(M, N):
    for K in ANY_K:
        if M * N * K > 6e9:
            continue
        print(f"ragged linear M={M} K={K} N={N}", flush=True)
        x, w, b = si.make_inputs((M, K, N), seed=M + 3 * K + 7 * N, dist="student_t")
        wq_o, sw_o = oracle.quantize_rows(w)
        y_o, xq_o, sx_o, acc_o = oracle.linear(x, wq_o, sw_o, b)
        wq, sw = w8a8.quantize_weight(dev_bf16(w))
        assert np.array_equal(wq.cpu().numpy(), wq_o) and np.array_equal(sw.cpu().numpy(), sw_o)
        xq, sx = w8a8.quantize_act(dev_bf16(x))
        assert np.array_equal(xq.cpu().numpy(), xq_o) and np.array_equal(sx.cpu().numpy(), sx_o)
        assert np.array_equal(w8a8.gemm_acc_i32(xq, wq).cpu().numpy(), acc_o), (M, N, K)
        y = w8a8.linear(dev_bf16(x), wq, sw, dev_bf16(b))
        assert_bf16_parity(host_bits(y), y_o, f"ragged {M}x{K}x{N}")


@pytest.mark.parametrize("ox,ow,oy", [(1, 0, 0), (0, 3, 0), (8, 4, 1), (5, 2, 3)])
def test_any_alignment_pointers(ox, ow, oy):
    """K % 16 == 0 and N % 8 == 0 at unaligned addresses, and every residue of the output
    rows; the bytes around the output stay as they were."""
    for M, N, K in [(7, 128, 256), (70, 264, 1040), (300, 520, 384)]:
        x, w, b = si.make_inputs((M, K, N), seed=M + K + N + ox)
        wq_o, sw_o = oracle.quantize_rows(w)
        y_o, xq_o, sx_o, _ = oracle.linear(x, wq_o, sw_o, b)
        xq = at_offset(torch.from_numpy(xq_o).cuda(), ox)
        wq = at_offset(torch.from_numpy(wq_o).cuda(), ow)
        sx, sw = torch.from_numpy(sx_o).cuda(), torch.from_numpy(sw_o).cuda()
        buf = torch.full((M * N + oy + 64,), 1.5, dtype=torch.bfloat16, device="cuda")
        y = buf[oy:oy + M * N].view(M, N)
        w8a8.gemm(xq, sx, wq, sw, dev_bf16(b), out=y)
        assert_bf16_parity(host_bits(y), y_o, f"offsets {ox},{ow},{oy} {M}x{K}x{N}")
        assert (buf[:oy] == 1.5).all() and (buf[oy + M * N:] == 1.5).all()


@pytest.mark.parametrize("N", [1, 7, 9, 250, 255, 257, 1001])
def test_ragged_channels_every_tile(N):
    """Aligned operands, output rows at every alignment: each tile's staged epilogue stores
    16 bytes at the row's own alignment and the last chunk element by element."""
    M, K = 97, 144
    x, w, b = si.make_inputs((M, K, N), seed=N)
    wq_o, sw_o = oracle.quantize_rows(w)
    y_o, xq_o, sx_o, _ = oracle.linear(x, wq_o, sw_o, b)
    xq, wq = torch.from_numpy(xq_o).cuda(), torch.from_numpy(wq_o).cuda()
    sx, sw = torch.from_numpy(sx_o).cuda(), torch.from_numpy(sw_o).cuda()
    for tile in range(w8a8.tile_count()):
        buf = torch.full((M * N + 64,), 1.5, dtype=torch.bfloat16, device="cuda")
        y = buf[:M * N].view(M, N)
        w8a8.gemm(xq, sx, wq, sw, dev_bf16(b), tile=tile, out=y)
        assert_bf16_parity(host_bits(y), y_o, f"tile {tile} N={N}")
        assert (buf[M * N:] == 1.5).all(), tile
