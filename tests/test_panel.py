"""33 to 128 activation rows without a plan: one launch (panel_kernel).  Against the oracle at the edges of its tiles --
blocks of 32 rows, panels of 32 and 64 channels times two, K parts without a tile, K slices -- with the bars of
test_gpu_parity (per element: half a 16-bit ulp plus 1e-5 of the sum of magnitudes for the fp32 accumulation)."""
import numpy as np
import pytest

import lutq_inputs as gen
from gpu_util import DeviceCase, to_bits, to_dev
from oracle import lutq_oracle as orc
from test_gpu_parity import check_y, tk

pytestmark = pytest.mark.gpu

# (M, row blocks, K tiles, group): one K tile for four parts and a lone row block; panels cut by the last row block; scale rows
# that are not whole 16-byte units (the scales go tile by tile) and ones that are (eight at a time); uneven K slices; two
# super-block sizes (257..512 row blocks); the taller panel with and without slices (from its fitted choice); an odd number
# of super-blocks of one
EDGES = [(33, 1, 1, 32), (64, 3, 2, 128), (65, 4, 3, 64), (96, 5, 4, 32), (97, 13, 5, 128), (128, 21, 8, 64),
         (128, 8, 9, 32), (50, 257, 4, 64), (128, 300, 8, 128), (100, 64, 33, 32), (80, 128, 16, 256), (34, 640, 6, 64),
         (128, 1024, 4, 128),
         # parts of M: small matrices, the last part of one row, of 32, or (M = 65 above) all but empty
         (65, 16, 32, 128), (97, 40, 8, 32), (128, 64, 4, 64), (72, 256, 2, 256), (128, 256, 8, 128)]


@pytest.mark.parametrize("bits", (4, 3, 2))
@pytest.mark.parametrize("dtype", ("f16", "bf16"))
def test_panel_matches_oracle(lutq, bits, dtype):
    workspace = None
    for i, (M, nb, kt, group) in enumerate(EDGES):
        K = kt * tk(bits)
        K += K % group
        c = gen.make_case(500 + i, M, 16 * nb, K, bits, group, dtype, ("nf", "learned", "random_index")[i % 3])
        d = DeviceCase(lutq, c)
        workspace = d.ws if workspace is None else workspace
        d.ws = workspace
        what = f"b{bits} {dtype} M{M} N{c.N} K{K} g{group}"
        Y = to_bits(d.matmul(lutq))
        check_y(Y, c, what)
        assert np.array_equal(Y, to_bits(d.matmul(lutq))), f"{what}: not reproducible"
        assert not workspace[:65536].any().item(), what


@pytest.mark.parametrize("op,bits,dim", (("lutq_matmul_pairs", 4, 2), ("lutq_matmul_quads", 2, 4)))
def test_panel_codebooks_and_static_scratch(lutq, op, bits, dim):
    """A codebook made of the scalar table, and the built-in scratch, give the call's own bits."""
    import torch
    for dtype in ("f16", "bf16"):
        for M, nb, kt in ((70, 9, 7), (128, 64, 16)):
            c = gen.make_case(900 + M, M, 16 * nb, kt * tk(bits), bits, 64, dtype, "learned")
            d = DeviceCase(lutq, c)
            want = to_bits(d.matmul(lutq))
            e = np.arange(256)
            book = to_dev(np.stack([c.T[(e >> (bits * j)) & ((1 << bits) - 1)] for j in range(dim)], axis=1), dtype)
            Y = torch.full((M, c.N), float("nan"), dtype=d.X.dtype, device="cuda")
            getattr(lutq, op)(d.X, d.packed, d.S, book, 64, Y, d.ws)
            assert np.array_equal(to_bits(Y), want)
            Y.fill_(float("nan"))
            lutq.lutq_matmul_static(d.X, d.packed, d.S, d.T, bits, 64, Y)
            assert np.array_equal(to_bits(Y), want)


def test_panel_rows_do_not_touch_each_other(lutq):
    """An infinity in the last activation row reaches that row alone, and rows beyond M are not written."""
    import torch
    c = gen.make_case(77, 41, 16 * 21, 2048, 4, 64, "f16", "learned")
    d = DeviceCase(lutq, c)
    want = to_bits(d.matmul(lutq))
    X = d.X.clone()
    X[40] = float("inf")
    Y = torch.full((128, c.N), 7.0, dtype=X.dtype, device="cuda")
    lutq.lutq_matmul(X, d.packed, d.S, d.T, 4, 64, Y[:41], d.ws)
    assert np.array_equal(to_bits(Y[:40]), want[:40])
    assert not torch.isfinite(Y[40]).any().item() and (Y[41:] == 7.0).all().item()


def test_panel_graph_replays_match_eager(lutq):
    """Captured with K slices (counters and partial sums in the workspace), replayed with eager calls between."""
    import torch
    for M, nb, kt in ((64, 64, 32), (128, 320, 16)):
        c = gen.make_case(40 + M, M, 16 * nb, kt * 128, 4, 128, "f16", "nf")
        d = DeviceCase(lutq, c)
        want = to_bits(d.matmul(lutq))
        check_y(want, c, f"M{M}")
        Y = torch.zeros((M, c.N), dtype=d.X.dtype, device="cuda")
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            lutq.lutq_matmul(d.X, d.packed, d.S, d.T, 4, 128, Y, d.ws)
        for _ in range(6):
            Y.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert np.array_equal(to_bits(Y), want)
            assert np.array_equal(to_bits(d.matmul(lutq)), want)


def test_registered_and_given_plans_keep_the_slices(lutq):
    """A plan given, or registered for slices of 32 rows, is what runs: the bits are those of the slices."""
    c = gen.make_case(3, 96, 16 * 24, 2048, 4, 64, "f16", "nf")
    d = DeviceCase(lutq, c)
    plan = lutq.Plan(1, 5, 8, 2, 1)
    sliced = to_bits(d.matmul(lutq, plan=plan))
    check_y(sliced, c, "slices")
    parts = np.concatenate([to_bits(d.matmul(lutq, plan=plan, X=d.X[i:i + 32].contiguous())) for i in (0, 32, 64)])
    assert np.array_equal(sliced, parts)
    try:
        lutq.lutq_plan_table_set([(4, 64, 0, 1, 32, c.N, c.K, plan)])
        assert np.array_equal(to_bits(d.matmul(lutq)), sliced)
    finally:
        lutq.lutq_plan_table_set([])
    check_y(to_bits(d.matmul(lutq)), c, "one launch")
