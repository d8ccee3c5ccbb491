"""The host side of the default plan: what it asks of the caller, and the rules of its cost
model (no GPU needed, except where marked)."""
import os
import re

import numpy as np
import pytest

import paper_2606_14598_amd as w8a8

# Sizes that only the any-alignment kernels run: K % 4 != 0, or K % 16 != 0 up to 32 tokens.
ANY_ALIGNMENT = [(64, 4096, 8193), (20, 4096, 8200), (100, 8000, 8193), (32, 2049, 16388),
                 (33, 4096, 8194), (128, 100, 133143), (512, 4608, 53247), (1, 1, 1)]


@pytest.mark.parametrize("M,N,K", ANY_ALIGNMENT)
def test_any_alignment_sizes_need_no_partials(M, N, K):
    """Those kernels never split K, so neither the query nor the least may ask for
    partials, whichever tile is given."""
    lib = w8a8.load_library()
    for tile in range(-1, w8a8.tile_count()):
        assert w8a8.gemm_workspace_bytes(M, N, K, tile) == 0, tile
    assert lib.w8a8_gemm_workspace_least_bytes(M, N, K) == 0
    head = -(-M * K // 256) * 256 + -(-4 * M // 256) * 256     # Xq and sx
    assert w8a8.linear_workspace_bytes(M, N, K) == head
    assert lib.w8a8_linear_workspace_least_bytes(M, N, K) == head


def test_default_plan_says_what_runs():
    """The query agrees with the workspace that the same plan asks for, names the kernels
    that are no tiles, and rejects what the GEMM rejects."""
    seen = set()
    for M in (1, 2, 8, 16, 17, 33, 64, 128, 129, 333, 512, 640, 2560, 4608):
        for N in (128, 1000, 4096, 4608, 16384):
            for K in (256, 1000, 1004, 1001, 4096, 8200, 16384, 53248):
                tile, splits = w8a8.default_plan(M, N, K)
                seen.add(min(tile, 0))
                partials = splits * M * N * 4 if splits > 1 else 0
                assert w8a8.gemm_workspace_bytes(M, N, K) == partials, (M, N, K)
                any_only = K % 4 != 0 or (K % 16 != 0 and M <= 32)
                if any_only:
                    assert tile == w8a8.PLAN_ANY, (M, N, K)
                if tile == w8a8.PLAN_ROWS:
                    assert M <= 8 and K % 16 == 0
                if tile >= 0:
                    name = w8a8.tile_name(tile)
                    assert not re.search(r"_k\d+$", name)
                    assert w8a8.plan_name(M, N, K) == name + (f"_k{splits}" if splits > 1 else "")
    assert seen == {0, w8a8.PLAN_ROWS, w8a8.PLAN_ANY}
    assert w8a8.plan_name(512, 4608, 53248) == "m256n256k64w2x4s4_k7"
    assert w8a8.plan_name(1, 4096, 4096) == "rows"
    for bad in ((0, 8, 8), (8, 0, 8), (8, 8, -1), (8, 8, w8a8.MAX_K + 1)):
        assert w8a8.default_plan(*bad) == (-1, 1)


@pytest.mark.parametrize("M", [5, 8])
def test_row_kernel_at_five_to_eight_tokens(M):
    """Only where it beats the tile that ran before it: on 16384 channels and more with a
    weight of 32 MB."""
    for N, K in ((16384, 2048), (16384, 4096), (20480, 2048)):
        assert w8a8.plan_name(M, N, K) == "rows", (N, K)
    for N, K in ((12288, 4096), (16383, 4096), (12288, 3072), (16384, 2032), (20480, 1024)):
        assert w8a8.plan_name(M, N, K) != "rows", (N, K)
    assert w8a8.plan_name(4, 12288, 4096) == "rows"


def test_sizes_beside_them_keep_their_partials():
    assert w8a8.gemm_workspace_bytes(64, 4096, 8192) > 0
    assert w8a8.gemm_workspace_bytes(33, 640, 24572) > 0


def _tile_table():
    """(costs by tile id, entries (m_lo, m_hi, N, K, tile)) of tile_table.inc."""
    path = os.path.join(os.path.dirname(w8a8.__file__), "csrc", "tile_table.inc")
    text = open(path).read()
    costs = text[text.index("kTileCost[] = {"):]
    costs = re.findall(r"\{([-0-9.e+]+), ([-0-9.e+]+)\}", costs[:costs.index("};")])
    entries = re.findall(r"\{(\d+), (\d+), (\d+), (\d+), (\d+)\}", text)
    return ([(float(c), float(d)) for c, d in costs], [tuple(map(int, e)) for e in entries])


def test_k_is_split_only_where_the_best_unsplit_tile_takes_over_12_us():
    """Over the table's shapes (above 128 tokens, where every unsplit candidate is in the
    wave cost model) and random ones without an entry."""
    costs, entries = _tile_table()
    names = [w8a8.tile_name(i) for i in range(w8a8.tile_count())]
    dims = [re.match(r"m(\d+)n(\d+)", n) for n in names]
    dims = [m and (int(m[1]), int(m[2])) for m in dims]

    def unsplit_us(M, N, K):
        return min(1e3 * -(-(-(-M // tm) * -(-N // tn)) // 256) * (c + d * 1e-9 * tm * tn * K)
                   for (c, d), (tm, tn) in ((costs[i], dims[i]) for i in range(len(names))
                                            if costs[i][1] > 0))
    rng = np.random.default_rng(5)
    shapes = {(M, N, K) for lo, hi, N, K, _ in entries
              for M in (lo, (lo + min(hi, 9000)) // 2, min(hi, 9000)) if 128 < M <= 9000}
    shapes |= {(int(2 ** rng.uniform(7.1, 12)), int(2 ** rng.uniform(7, 13)),
                int(2 ** rng.uniform(8, 14.6)) // 16 * 16) for _ in range(2000)}
    split = 0
    for M, N, K in sorted(shapes):
        if w8a8.gemm_workspace_bytes(M, N, K) > 0:
            split += 1
            assert unsplit_us(M, N, K) > 12.0, (M, N, K)
    assert split > 50


def test_a_split_has_to_be_predicted_clearly_faster():
    """Shapes where a split predicted up to 5% faster ran 3-7% slower than the unsplit tile."""
    for M, N, K in ((160, 4096, 8192), (333, 4096, 8192), (96, 4096, 4096)):
        assert w8a8.default_plan(M, N, K)[1] == 1, (M, N, K)
    assert w8a8.plan_name(512, 4608, 53248) == "m256n256k64w2x4s4_k7"


def test_cost_rows_stand_at_their_tiles():
    """The costs are matched to the tiles by position (kTileCost) or id (kStreamCost): the
    tile that a row was fitted for is the one named beside it."""
    path = os.path.join(os.path.dirname(w8a8.__file__), "csrc", "tile_table.inc")
    text = open(path).read()
    rows = text[text.index("kTileCost[] = {"):text.index("kStreamCost[] = {")]
    names = re.findall(r"\},  // (\w+)", rows)
    assert names == [w8a8.tile_name(i) for i in range(w8a8.tile_count())]
    rows = text[text.index("kStreamCost[] = {"):text.index("kTileTable[]")]
    ids = re.findall(r"\{(\d+), [^}]*\},  // (\w+)", rows)
    assert [w8a8.tile_name(int(i)) for i, _ in ids] == [name for _, name in ids]
    assert {n for _, n in ids} == {n for n in names if n.startswith(("skinny", "wsx"))}


def test_token_block_tiles_only_where_the_block_fits_in_lds():
    """Above 16 tokens the plan takes a tile that keeps its token block in LDS only where it
    does (elsewhere that id runs another kernel, which the tile's cost does not describe),
    and does take it where it was measured fastest (33 to 64 tokens)."""
    from paper_2606_14598_amd.tune import stream_fits
    for M, N, K in ((64, 4096, 4096), (40, 3072, 3072), (33, 3072, 3072), (56, 4096, 4096)):
        assert w8a8.plan_name(M, N, K) == "wsx_m32n32w8d2", (M, N, K)
    rng = np.random.default_rng(3)
    seen = 0
    for _ in range(3000):
        M, N = int(rng.integers(17, 129)), int(2 ** rng.uniform(7, 14))
        K = int(2 ** rng.uniform(8, 14.6)) // 16 * 16
        name = w8a8.plan_name(M, N, K)
        if name.startswith("wsx"):
            seen += 1
            assert stream_fits(name, M, K), (M, N, K, name)
    assert seen > 300


def test_fit_recovers_the_costs_of_a_synthetic_sweep():
    from paper_2606_14598_amd import tune
    names = [w8a8.tile_name(i) for i in range(w8a8.tile_count())]
    rng = np.random.default_rng(7)
    stream = [n for n in names if n.startswith(("skinny", "wsx"))]
    tiles = [n for n in names if n not in tune.UNMODELED and n not in stream
             and not re.search(r"_k\d+$", n)]
    want = {n: rng.uniform(0.5, 2, 8) * [3, 1, 1, 1, .05, .05, .05, .2] for n in stream}
    want |= {n: rng.uniform(0.5, 2, 2) * [5e-3, 0.2] for n in tiles}
    import random
    r, rows = random.Random(1), []
    for i in range(400):
        M, N, K = tune.random_shape(r, 128 if i % 2 else 8192)
        assert 17 <= M <= 8192 and K % 16 == 0 and N % 16 == 0
        us = {n: float(np.dot(want[n], tune.cost_terms(n, M, N, K))) for n in tiles}
        if M <= 128:
            # a token block that does not fit runs another kernel: it must not be fitted
            us |= {n: float(np.dot(want[n], tune.cost_terms(n, M, N, K)))
                   * (1 if tune.stream_fits(n, M, K) else 3) for n in stream}
        rows.append({"M": M, "N": N, "K": K, "us": us})
    got = tune.fit_costs(rows, names)
    assert set(got) == set(want)
    for n in want:
        for row in rows[::7]:
            M, N, K = row["M"], row["N"], row["K"]
            if n in row["us"] and (n in tiles or tune.stream_fits(n, M, K)):
                t = float(np.dot(got[n], tune.cost_terms(n, M, N, K)))
                assert abs(t / row["us"][n] - 1) < 1e-6, n


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(64, 1000, 8193), (20, 4096, 8200)])
def test_any_alignment_gemm_without_a_workspace(M, N, K):
    import torch
    import oracle
    import synth_inputs as si
    from _helpers import dev_bf16, host_bits, say
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lib = w8a8.load_library()
    say(f"no workspace M={M} N={N} K={K}")
    x, w, b = si.make_inputs((M, K, N), seed=M + K)
    wq_o, sw_o = oracle.quantize_rows(w)
    y_o, xq_o, sx_o, _ = oracle.linear(x, wq_o, sw_o, b)
    xq, sx = w8a8.quantize_act(dev_bf16(x))
    wq, sw = w8a8.quantize_weight(dev_bf16(w))
    bd = dev_bf16(b)
    y = torch.empty(M, N, dtype=torch.bfloat16, device="cuda")
    st = lib.w8a8_gemm(xq.data_ptr(), sx.data_ptr(), wq.data_ptr(), sw.data_ptr(),
                       bd.data_ptr(), y.data_ptr(), M, N, K, None, 0,
                       torch.cuda.current_stream().cuda_stream)
    assert st == 0, lib.w8a8_status_string(st)
    assert np.array_equal(host_bits(y), y_o)
