"""One table per output row on the row-streaming kernel, 5 to 32 rows: four and eight row blocks side by side, K slices, scale
rows that are not whole 16-byte units, one reduction round over the table's own area -- against the oracle, with the bars of
test_gpu_parity (per element: half a 16-bit ulp plus 1e-5 of the sum of magnitudes for the fp32 accumulation)."""
import numpy as np
import pytest

import lutq_inputs as gen
from gpu_util import DeviceCase, to_bits, to_dev
from oracle import lutq_oracle as orc
from test_gpu_parity import check_y, tk

# (M, row blocks, K tiles, group): five to eight row blocks per compute unit (one pass of eight, the last short), nine (two
# passes), two and four (passes of four), between one and two, a lone one and a few with many slices, slices of one tile
SHAPES = [(5, 1280, 2, 128), (16, 1793, 1, 64), (17, 2048, 2, 128), (32, 1400, 1, 32), (16, 2304, 1, 128), (8, 512, 4, 64),
          (32, 1024, 2, 256), (12, 300, 4, 64), (17, 257, 3, 128), (32, 511, 4, 256), (17, 1, 64, 128), (30, 13, 64, 64),
          (17, 82, 67, 128), (25, 128, 48, 32), (16, 37, 88, 256), (10, 64, 90, 64)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("bits", [4, 3, 2])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "m%d_nb%d_kt%d_g%d" % s)
def test_row_tables(shape, bits, dtype):
    import torch
    import paper_2407_10960_amd as lutq
    M, nb, kt, group = shape
    if bits != 4:
        kt = (kt + 1) // 2
    N, K = 16 * nb, tk(bits) * kt
    if K % group:
        K *= 2
    case = gen.make_case(17 * M + nb + bits, M, N, K, bits, group, dtype, "random_index")
    d = DeviceCase(lutq, case)
    rng = np.random.default_rng(nb + kt)
    tables = gen.encode16(rng.standard_normal((N, 1 << bits)), dtype)
    Y = torch.full((M, N), float("nan"), dtype=d.X.dtype, device="cuda")
    for _ in range(2):                       # (the counters are zero again for the second call)
        lutq.lutq_matmul_channel(d.X, d.packed, d.S, to_dev(tables, dtype), bits, group, Y, d.ws)
    torch.cuda.synchronize()
    What = orc.dequant_channel(case.Q, tables, case.S, group, dtype)
    check_y(to_bits(Y), case, f"{shape} b{bits} {dtype}", What)
    assert not d.ws[:65536].any().item()


# (bits, group, M, N, K, dtype), what is launched
LAUNCHED = [((3, 32, 11, 80, 17408, 1), "slices"), ((4, 32, 12, 64, 13312, 0), "slices"), ((3, 64, 9, 16, 29440, 0), "slices"),
            ((3, 32, 25, 64, 22528, 1), "slices"), ((2, 256, 30, 48, 12288, 0), "slices"),
            ((4, 128, 10, 7312, 1536, 1), "teams"), ((4, 128, 11, 5152, 1920, 1), "teams"), ((3, 64, 6, 33264, 3840, 1), "teams"),
            ((4, 32, 5, 18304, 1920, 1), "teams"), ((4, 32, 5, 20560, 1920, 1), "rows"), ((4, 32, 5, 18304, 1920, 0), "teams"), ((4, 32, 7, 18304, 1920, 0), "rows"),
            ((3, 64, 6, 33696, 5376, 0), "teams"), ((2, 128, 8, 18896, 7936, 1), "teams"), ((4, 64, 6, 33808, 5760, 1), "teams"), ((4, 64, 7, 33808, 5760, 1), "rows"),
            ((3, 32, 9, 3600, 11520, 1), "teams"), ((3, 32, 11, 3600, 11520, 1), "slices"), ((3, 32, 10, 2560, 11520, 1), "slices"),
            ((4, 32, 19, 5968, 1152, 0), "teams"), ((4, 32, 23, 5968, 1152, 0), "slices"), ((4, 32, 19, 5968, 2048, 0), "slices"), ((4, 32, 19, 5968, 1152, 1), "slices"),
            ((4, 128, 12, 4800, 5632, 0), "rows"), ((3, 128, 16, 7264, 2048, 1), "rows"), ((4, 64, 6, 33264, 3840, 0), "rows")]


def test_launches_with_one_table_per_row():
    """At most sixteen K slices; four-bit calls of 9..16 rows with one to two row blocks per compute unit and a short K, and 3-bit bf16
    calls of five and six rows with scale rows that are not whole 16-byte units, stay with the teams; so do 5..8 rows with such scale
    rows that end in a pass of one row block, and two classes of K slices."""
    import paper_2407_10960_amd as lutq
    for p, what in LAUNCHED:
        plan = lutq.calib_plan(*p, row_tables=True)
        assert plan.scheduling == (1 if what == "teams" else 3), (p, plan)
        assert (what == "slices") == (plan.tiles_per_item > 0), (p, plan)
    rng = np.random.default_rng(1)
    for _ in range(2000):
        bits, group, M = int(rng.choice([2, 3, 4])), int(rng.choice([32, 64, 128, 256])), int(rng.integers(5, 33))
        N, K = 16 * int(np.exp(rng.uniform(0, 7))), 256 * int(rng.integers(16, 128))
        plan = lutq.calib_plan(bits, group, M, N, K, int(rng.integers(0, 2)), row_tables=True)
        if plan.tiles_per_item:
            shares = -(-(N // 16) // 4)
            assert plan.grid % shares == 0 and 2 <= plan.grid // shares <= 16, (bits, group, M, N, K, plan)
