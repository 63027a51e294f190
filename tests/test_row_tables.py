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
