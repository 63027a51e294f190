"""33 to 128 activation rows without a plan: one launch (panel_kernel).  Against the oracle at the edges of its tiles --
blocks of 32 rows, panels of 32 and 64 channels times two, K parts without a tile, K slices -- with the bars of
test_gpu_parity (per element: half a 16-bit ulp plus 1e-5 of the sum of magnitudes for the fp32 accumulation)."""
import numpy as np
import pytest

import lutq_inputs as gen
from gpu_util import DeviceCase, to_bits, to_dev
from oracle import lutq_oracle as orc
from test_gpu_parity import check_y, tk

# (M, row blocks, K tiles, group): one K tile for four parts and a lone row block; panels cut by the last row block; scale rows
# that are not whole 16-byte units (the scales go tile by tile) and ones that are (eight at a time); uneven K slices; two
# super-block sizes (257..512 row blocks); an odd number of super-blocks of one
EDGES = [(33, 1, 1, 32), (64, 3, 2, 128), (65, 4, 3, 64), (96, 5, 4, 32), (97, 13, 5, 128), (128, 21, 8, 64),
         (128, 8, 9, 32), (50, 257, 4, 64), (128, 300, 8, 128), (100, 64, 33, 32), (80, 128, 16, 256), (34, 640, 6, 64),
         (128, 1024, 4, 128),
         # parts of M: small matrices, the last part of one row, of 32, or (M = 65 above) all but empty
         (65, 16, 32, 128), (97, 40, 8, 32), (128, 64, 4, 64), (72, 256, 2, 256), (128, 256, 8, 128)]


# One case per instance of the kernel that the choice reaches, each with and without K slices and with scales eight at a time and
# tile by tile (a class: blocks of 32 rows, panel height / 32, slices, scales eight at a time); (M, row blocks, K tiles, group)
CLASSES = {
    4: [(33, 1, 1, 32), (33, 1, 2, 32), (50, 1, 12, 256), (33, 1, 12, 32), (65, 600, 1, 64), (66, 600, 2, 32), (96, 200, 33, 32),
        (90, 200, 48, 64), (97, 257, 1, 32), (120, 257, 2, 32), (97, 96, 33, 128), (128, 96, 40, 32), (100, 600, 1, 128),
        (97, 600, 2, 32), (97, 257, 33, 64), (128, 257, 40, 128), (65, 768, 1, 32), (80, 768, 2, 32), (65, 200, 40, 256),
        (96, 200, 40, 128), (65, 1280, 1, 32), (96, 1280, 2, 32), (70, 384, 64, 128), (97, 1280, 1, 64), (128, 1280, 2, 32),
        (100, 257, 112, 256)],
    3: [(33, 1, 1, 256), (64, 1, 1, 32), (40, 1, 9, 128), (33, 1, 8, 32), (65, 128, 20, 256), (96, 128, 20, 64), (97, 257, 1, 128),
        (128, 257, 1, 32), (97, 96, 12, 256), (100, 96, 12, 32), (33, 1280, 1, 64), (64, 1280, 1, 32), (50, 384, 33, 256),
        (33, 384, 33, 32), (65, 600, 1, 256), (90, 600, 1, 32), (65, 160, 20, 256), (96, 160, 20, 128), (65, 1280, 1, 128),
        (96, 1280, 1, 32), (65, 384, 33, 64), (80, 384, 33, 32), (97, 600, 1, 256), (128, 600, 1, 32), (128, 200, 33, 256),
        (97, 257, 24, 128)],
    2: [(33, 1, 1, 256), (64, 1, 1, 32), (40, 1, 9, 128), (33, 1, 8, 32), (65, 600, 1, 64), (96, 600, 1, 32), (65, 128, 20, 256),
        (90, 128, 20, 64), (97, 257, 1, 128), (128, 257, 1, 32), (97, 96, 20, 256), (100, 96, 20, 32), (97, 600, 1, 128),
        (128, 600, 1, 32), (97, 200, 33, 256), (97, 257, 24, 32), (65, 768, 1, 256), (96, 768, 1, 32), (65, 256, 33, 64),
        (80, 96, 64, 128), (65, 1280, 1, 256), (96, 1280, 1, 32), (70, 384, 33, 64), (65, 384, 33, 32), (97, 1280, 1, 64),
        (128, 1280, 1, 32), (100, 600, 33, 256), (97, 600, 24, 32)],
}


def route_class(lutq, bits, dtype, M, nb, kt, group):
    """The class of a call's launch, None where it is served in slices."""
    K = kt * tk(bits)
    r = lutq.calib_route(bits, group, M, 16 * nb, K, 0 if dtype == "f16" else 1)
    return None if r[0] else (r[1], r[2], r[3] > 1, K // group * 2 % 16 == 0)


@pytest.mark.parametrize("bits", (4, 3, 2))
@pytest.mark.parametrize("dtype", ("f16", "bf16"))
def test_cases_reach_every_instance_the_choice_reaches(lutq, bits, dtype):
    """CLASSES names every class that shapes up to 3584 row blocks, 128 K tiles and 128 rows lead to, and EDGES is served by
    one launch (host logic, 256 compute units)."""
    reached = set()
    for M in (33, 64, 65, 96, 97, 128):
        for nb in (1, 2, 3, 5, 8, 13, 16, 24, 32, 48, 64, 96, 128, 160, 200, 256, 257, 300, 384, 448, 512, 600, 640, 768, 1024, 1280,
                   1792, 2048, 2560, 3584):
            for kt in (1, 2, 3, 4, 8, 9, 12, 16, 20, 24, 32, 33, 40, 48, 64, 80, 112, 128):
                for group in (32, 64, 256):
                    if kt * tk(bits) % group == 0 and 16 * nb * kt * tk(bits) * bits < 1 << 34:
                        reached.add(route_class(lutq, bits, dtype, M, nb, kt, group))
    covered = [route_class(lutq, bits, dtype, *case) for case in CLASSES[bits]]
    assert None not in covered and len(set(covered)) == len(covered)
    assert reached - {None} == set(covered)
    for M, nb, kt, group in EDGES:
        K = kt * tk(bits)
        kt = (K + K % group) // tk(bits)
        assert route_class(lutq, bits, dtype, M, nb, kt, group) is not None, (M, nb, kt, group)


@pytest.mark.gpu
@pytest.mark.parametrize("bits", (4, 3, 2))
@pytest.mark.parametrize("dtype", ("f16", "bf16"))
def test_every_instance_matches_oracle(lutq, bits, dtype):
    """All rows of 160 sampled weight rows, first and last row blocks included, of every class."""
    workspace, rng = None, np.random.default_rng(bits)
    for i, (M, nb, kt, group) in enumerate(CLASSES[bits]):
        N = 16 * nb
        c = gen.make_case(700 + i, M, N, kt * tk(bits), bits, group, dtype, "random_index")
        d = DeviceCase(lutq, c)
        workspace = d.ws if workspace is None else workspace
        d.ws = workspace
        what = f"b{bits} {dtype} M{M} N{N} K{c.K} g{group}"
        print(what, flush=True)
        Y = to_bits(d.matmul(lutq))
        rows = np.arange(N) if N <= 160 else np.unique(np.concatenate([np.arange(16), np.arange(N - 16, N), rng.choice(N, 128, replace=False)]))
        check_y(Y[:, rows], gen.Case(M, len(rows), c.K, bits, group, dtype, c.X, c.Q[rows], c.S[rows], c.T), what)
        assert np.isfinite(orc.to_f64(Y, dtype)).all(), what
        assert np.array_equal(Y, to_bits(d.matmul(lutq))), f"{what}: not reproducible"
        assert not workspace[:65536].any().item(), what


@pytest.mark.gpu
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


@pytest.mark.gpu
@pytest.mark.parametrize("op,bits,dim", (("lutq_matmul_pairs", 4, 2), ("lutq_matmul_quads", 2, 4)))
def test_panel_codebooks_and_static_scratch(lutq, op, bits, dim):
    """A codebook made of the scalar table, and the built-in scratch, give the call's own bits; also where row streaming is the
    faster launch (12288 x 4096, 48 rows)."""
    import torch
    assert lutq.calib_route(4, 64, 48, 12288, 4096, 0)[0] == lutq.calib_route(4, 64, 48, 12288, 4096, 1)[0] == 64
    for dtype in ("f16", "bf16"):
        for M, nb, kt in ((70, 9, 7), (128, 64, 16), (48, 768, 32 if bits == 4 else 4)):
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


@pytest.mark.gpu
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


@pytest.mark.gpu
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


@pytest.mark.gpu
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


def test_only_a_registered_plan_that_can_run_keeps_the_slices(lutq):
    """Routes of calls of 33..128 rows with plans registered for up to 32 rows (host logic, 256 compute units)."""
    def route(plan, bits, N, K, M=96, m_max=32, ws=None):
        try:
            lutq.lutq_plan_table_set([(bits, 128, 0, 1, m_max, N, K, plan)])
            return lutq.calib_route(bits, 128, M, N, K, 0, 256, ws)[0]
        finally:
            lutq.lutq_plan_table_set([])
    decode = lutq.Plan(1, 256, 12, 2, 7, 2, 4)
    team = lutq.Plan(1, 128, 8, 2, 1)
    assert route(team, 4, 2048, 4096) == 32 and route(team, 3, 28672, 4096) == 32        # slices of 32 rows that run it
    assert route(team, 4, 28672, 4096, 128) == 0                # its slices are of 64 rows, which take no plan from the table
    assert route(decode, 4, 2048, 4096) == 0                    # a work queue is for up to four rows
    assert route(lutq.Plan(1, 0, 8, 2, 3), 4, 2048, 4096) == 0                           # eight waves are not three teams
    assert route(team, 4, 2048, 4096, m_max=16) == 0 and route(lutq.Plan(), 4, 2048, 4096) == 0
    # 64 MiB of partial sums fit a workspace and not the built-in scratch; so do a row-streaming plan's slices
    for plan in (lutq.Plan(4, 4095, 4, 2, 1), lutq.Plan(8, 4096, 0, 2, 8, 3, 1)):
        assert lutq.lutq_plan_check(4, 128, 32, 2048, 32768, 0, 256, plan) == 0
        assert route(plan, 4, 2048, 32768) == 32 and route(plan, 4, 2048, 32768, ws=lutq.STATIC_SCRATCH_BYTES) == 0


@pytest.mark.gpu
def test_registered_plans_that_do_not_serve_a_call_leave_its_bits(lutq):
    for N, plan in ((4096, lutq.Plan(1, 128, 8, 2, 1)), (384, lutq.Plan(1, 0, 8, 2, 3))):
        c = gen.make_case(5, 100, N, 1024, 4, 64, "f16", "nf")
        d = DeviceCase(lutq, c)
        want = to_bits(d.matmul(lutq))
        try:
            lutq.lutq_plan_table_set([(4, 64, 0, 1, 32, c.N, c.K, plan)])
            assert np.array_equal(to_bits(d.matmul(lutq)), want)
        finally:
            lutq.lutq_plan_table_set([])
        check_y(want, c, f"N{N}")


@pytest.mark.gpu
def test_tuner_times_the_single_launch(lutq):
    """Beyond 32 rows the tuner's first candidate is the empty plan: 1024 x 4096 with 128 rows takes 9 us in one launch and 37
    in slices, so it is also what the tuner returns."""
    import torch
    M, N, K = 128, 1024, 4096
    c = gen.make_case(8, M, N, K, 4, 128, "f16", "nf")
    d = DeviceCase(lutq, c)
    cands = lutq.lutq_tune_candidates(4, 128, M, N, K, 0)
    assert cands[:2] == [lutq.Plan(), lutq.lutq_plan_default(4, 128, M, N, K, 0)] and len(set(map(repr, cands))) == len(cands)
    Y = torch.empty((M, N), dtype=torch.float16, device="cuda")
    plan, us = lutq.lutq_tune(d.X, [d.packed, d.packed.clone()], [d.S, d.S.clone()], d.T, 4, 128, Y, d.ws, reps=5)
    assert plan == lutq.Plan() and us > 0.5
    want = to_bits(d.matmul(lutq))
    assert np.array_equal(to_bits(d.matmul(lutq, plan=plan)), want)
    try:                                            # registered, it leaves the call as it is
        lutq.lutq_plan_table_set([(4, 128, 0, 1, 128, N, K, plan)])
        assert np.array_equal(to_bits(d.matmul(lutq)), want)
    finally:
        lutq.lutq_plan_table_set([])


def test_row_streaming_keeps_a_call_only_where_its_launch_exists(lutq):
    """4 bits, up to 64 rows: scale rows too long for the LDS of that launch, or a copy of the activations that does not fit the
    scratch, leave the call to the panel kernel (slices of 32 rows, or none at all, would be what is left)."""
    for M, N, K, group in ((40, 10240, 28672, 32), (33, 12288, 24576, 32), (48, 12288, 32768, 32)):
        assert lutq.lutq_plan_default_for(4, group, M, N, K, 0, 256).scheduling != 3
        assert lutq.calib_route(4, group, M, N, K, 0)[0] == 0
    for M in (33, 48):
        K = 180224                                   # 16.5 MiB and more of activations
        assert lutq.calib_route(4, 64, M, 10240, K, 0, 256, lutq.STATIC_SCRATCH_BYTES)[0] == 0


# (type, M, N, K, row streaming us, panel us), group 128, HBM-cold weights: pairs that differ by 8 % and more
MEASURED_W4 = [
    ("f16", 40, 4096, 4096, 13.0, 11.7), ("f16", 48, 5120, 5120, 16.3, 13.4), ("f16", 33, 6144, 4096, 14.6, 13.5),
    ("f16", 64, 8192, 8192, 25.7, 21.6), ("f16", 64, 10240, 8192, 28.7, 25.2), ("f16", 40, 10240, 16384, 41.9, 37.4),
    ("f16", 48, 12288, 4096, 16.0, 17.5), ("f16", 64, 20480, 8192, 47.5, 41.5), ("f16", 48, 27648, 5120, 35.4, 30.4),
    ("f16", 40, 28672, 4096, 29.2, 24.6), ("f16", 33, 32768, 8192, 52.8, 47.9), ("f16", 48, 40960, 5120, 49.6, 55.7),
    ("f16", 64, 57344, 8192, 104.9, 94.2), ("bf16", 64, 4096, 4096, 15.5, 12.8), ("bf16", 33, 5120, 5120, 16.2, 13.9),
    ("bf16", 64, 6144, 4096, 17.6, 15.8), ("bf16", 48, 8192, 28672, 60.6, 53.2), ("bf16", 48, 10240, 8192, 24.8, 27.1),
    ("bf16", 40, 12288, 4096, 16.1, 18.8), ("bf16", 33, 12288, 12288, 34.6, 42.2), ("bf16", 48, 12288, 12288, 34.5, 42.5),
    ("bf16", 48, 16384, 6144, 24.7, 27.3), ("bf16", 40, 20480, 8192, 42.0, 48.9), ("bf16", 64, 28672, 4096, 34.8, 30.0),
    ("bf16", 33, 40960, 5120, 49.2, 63.5), ("bf16", 64, 40960, 5120, 58.3, 67.7), ("bf16", 40, 57344, 8192, 91.8, 105.2)]


def test_33_to_64_rows_at_4_bits_take_the_faster_launch(lutq):
    for dtype, M, N, K, rows_us, panel_us in MEASURED_W4:
        r = lutq.calib_route(4, 128, M, N, K, 0 if dtype == "f16" else 1)
        assert (r[0] == 0) == (panel_us < rows_us), (dtype, M, N, K, r)
