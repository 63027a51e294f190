"""Calls of up to 32 rows without a plan on shapes where the estimated times, not the rules, choose the launch: row streaming in
uneven K slices, with scale rows that are not whole 16-byte units, several passes, single teams, and every instance of the panel
kernel for one block of 32 rows that the choice reaches.  What each call launches is asked of the host logic (256 compute units)."""
import numpy as np
import pytest

import lutq_inputs as gen
import paper_2407_10960_amd as lutq
from gpu_util import DeviceCase, to_bits, to_dev
from oracle import lutq_oracle as orc
from test_gpu_parity import check_y, tk

# (bits, group, M, N, K, dtype): what is launched
LAUNCHES = {
    "row streaming in K slices": [(4, 256, 22, 1328, 23296, "bf16"), (4, 64, 13, 1248, 21504, "bf16"), (4, 128, 6, 4448, 11648, "bf16")],
    "row streaming": [(3, 64, 15, 8880, 4352, "bf16"), (4, 256, 12, 12304, 1536, "bf16"), (2, 64, 14, 14256, 3328, "bf16"),
                      (4, 256, 17, 26704, 1792, "f16"), (4, 64, 27, 9200, 3584, "bf16"), (3, 32, 18, 6000, 5376, "bf16")],
    "teams": [(4, 32, 2, 11536, 3968, "f16")],
    "the rules' plan": [(2, 32, 9, 21904, 1536, "bf16"), (3, 32, 9, 5072, 1536, "bf16"), (4, 64, 11, 10304, 1280, "f16"),
                        (3, 256, 10, 22672, 1536, "bf16"), (2, 32, 1, 19056, 1024, "f16"), (3, 64, 3, 9040, 2560, "bf16")],
    "panels": [(2, 64, 21, 1136, 13312, "f16"), (3, 32, 20, 2368, 4096, "f16"), (4, 32, 17, 1072, 22528, "f16"), (2, 32, 25, 2128, 12288, "bf16"),
               (3, 64, 32, 4272, 8192, "f16"), (2, 32, 32, 1152, 20992, "f16")]}
SHAPES = [s for shapes in LAUNCHES.values() for s in shapes]


def launch(bits, group, M, N, K, dtype):
    p = (bits, group, M, N, K, 0 if dtype == "f16" else 1)
    plan, route = lutq.calib_plan(*p), lutq.calib_route(*p)
    assert route[0] == 0 if plan == lutq.Plan() else route == (32, 0, 0, 0, 0)
    if plan == lutq.Plan():
        return "panels"
    if plan == lutq.lutq_plan_default_for(*p):
        return "the rules' plan"
    return "teams" if plan.scheduling == 1 else "row streaming in K slices" if plan.tiles_per_item else "row streaming"


def test_what_the_calls_launch():
    for what, shapes in LAUNCHES.items():
        assert [launch(*s) for s in shapes] == [what] * len(shapes)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "b%d_g%d_m%d_%dx%d_%s" % s)
def test_call_without_plan(shape):
    import torch
    bits, group, M, N, K, dtype = shape
    case = gen.make_case(N + M, M, N, K, bits, group, dtype, "random_index")
    d = DeviceCase(lutq, case)
    first = to_bits(d.matmul(lutq))
    check_y(first, case, str(shape))
    # the empty plan stands for none; that of lutq_plan_default means the rules' launch, also on the library's own scratch
    assert np.array_equal(first, to_bits(d.matmul(lutq, plan=lutq.Plan())))
    plan = lutq.lutq_plan_default(bits, group, M, N, K, 0 if dtype == "f16" else 1)
    ruled = to_bits(d.matmul(lutq, plan=plan))
    check_y(ruled, case, f"{shape} {plan}")
    Y = torch.full((M, N), float("nan"), dtype=d.X.dtype, device="cuda")
    lutq.lutq_matmul_static(d.X, d.packed, d.S, d.T, bits, group, Y, plan=plan)
    assert np.array_equal(ruled, to_bits(Y))
    Y = torch.full((M, N), float("nan"), dtype=d.X.dtype, device="cuda")
    lutq.lutq_matmul_static(d.X, d.packed, d.S, d.T, bits, group, Y)
    torch.cuda.synchronize()
    check_y(to_bits(Y), case, str(shape) + " static")
    assert not d.ws[:65536].any().item()


def test_every_call_without_plan_is_accepted():
    """Host logic: whatever the estimates choose can be launched, on devices of any size."""
    rng = np.random.default_rng(11)
    for i in range(3000):
        bits, group = int(rng.choice([2, 3, 4])), int(rng.choice([32, 64, 128, 256]))
        step = max(group, 128 if bits == 4 else 256)
        K = step * int(np.exp(rng.uniform(0, np.log(32768 / step))))
        N = 16 * int(np.exp(rng.uniform(0, np.log(6000))))
        M, dt, cus = int(rng.integers(1, 33)), int(rng.integers(0, 2)), int(rng.choice([256, 256, 304, 64, 8, 1]))
        if N * K * bits // 8 >= 1 << 31:
            continue
        assert lutq.lutq_plan_check(bits, group, M, N, K, dt, cus) == 0, (bits, group, M, N, K, dt, cus)


# Classes of the panel kernel's launches: panel height / 32, K slices, scales eight at a time.  (4-bit bf16: 64 channels in K slices
# with scales tile by tile is never the choice.)
CLASSES = [(rp, sliced, eight) for rp in (1, 2) for sliced in (False, True) for eight in (False, True)]
CANDIDATES = sorted(((M, nb, kt, group) for M in (17, 24, 32) for nb in (1, 3, 33, 96, 257, 384, 600, 1280, 1792)
                     for kt in (1, 2, 4, 8, 9, 12, 20, 33, 40, 64) for group in (32, 64, 256)), key=lambda c: (c[1] * c[2], c))


def panel_cases(bits, dtype):
    """For each class that is reached the candidate with the fewest weights."""
    found = {}
    for M, nb, kt, group in CANDIDATES:
        K = kt * tk(bits)
        if K % group == 0:
            r = lutq.calib_route(bits, group, M, 16 * nb, K, 0 if dtype == "f16" else 1)
            if r[0] == 0:
                assert r[1] == r[4] == 1
                found.setdefault((r[2], r[3] > 1, K // group % 8 == 0), (M, nb, kt, group))
    return found


@pytest.mark.parametrize("bits", (4, 3, 2))
@pytest.mark.parametrize("dtype", ("f16", "bf16"))
def test_every_panel_class_is_reached(bits, dtype):
    never = {(2, True, False)} if bits == 4 and dtype == "bf16" else set()
    assert set(panel_cases(bits, dtype)) == set(CLASSES) - never


@pytest.mark.gpu
@pytest.mark.parametrize("bits", (4, 3, 2))
@pytest.mark.parametrize("dtype", ("f16", "bf16"))
def test_every_panel_class_matches_oracle(bits, dtype):
    """All rows of up to 160 weight rows, first and last row blocks included; at 4 and 2 bits the scalar table as a codebook of pairs
    or quads gives the same bits."""
    import torch
    workspace, rng = None, np.random.default_rng(bits)
    for i, (M, nb, kt, group) in enumerate(panel_cases(bits, dtype).values()):
        N = 16 * nb
        c = gen.make_case(1700 + i, M, N, kt * tk(bits), bits, group, dtype, "random_index")
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
        if bits != 3:
            e, dim = np.arange(256), 2 if bits == 4 else 4
            book = to_dev(np.stack([c.T[(e >> (bits * j)) & ((1 << bits) - 1)] for j in range(dim)], axis=1), dtype)
            Z = torch.full((M, N), float("nan"), dtype=d.X.dtype, device="cuda")
            (lutq.lutq_matmul_pairs if bits == 4 else lutq.lutq_matmul_quads)(d.X, d.packed, d.S, book, group, Z, d.ws)
            assert np.array_equal(to_bits(Z), Y), what
        assert not workspace[:65536].any().item(), what
