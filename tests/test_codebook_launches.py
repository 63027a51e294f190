"""lutq_matmul_pairs (4-bit layout) and lutq_matmul_quads (2-bit layout) on every kernel that a call of up to 32 rows can take: the
scalar table as a codebook gives lutq_matmul's bits.  What each call launches is asked of the host logic (256 compute units)."""
import numpy as np
import pytest

import lutq_inputs as gen
from gpu_util import DeviceCase, to_bits, to_dev
from test_gpu_parity import check_y

QUEUE, ROWS = 2, 3
# (bits, group, M, N, K, dtype): scheduling (0: panels), row blocks side by side, K slices
CALLS = {(4, 64, 3, 112, 512, "f16"): (1, 1, False), (4, 32, 1, 4096, 512, "f16"): (QUEUE, 1, False),
         (4, 32, 8, 12288, 256, "bf16"): (ROWS, 4, False), (4, 32, 16, 24576, 256, "f16"): (ROWS, 8, False),
         (4, 32, 16, 48, 7168, "f16"): (ROWS, 4, True), (4, 64, 32, 48, 3584, "f16"): (ROWS, 4, True),
         (4, 32, 24, 24576, 256, "bf16"): (ROWS, 8, False), (4, 32, 32, 48, 2560, "f16"): (0, 0, False),
         (2, 64, 3, 112, 512, "bf16"): (1, 1, False), (2, 32, 1, 8192, 1024, "f16"): (QUEUE, 1, False),
         (2, 32, 16, 4112, 2048, "f16"): (ROWS, 4, False), (2, 64, 6, 20560, 2048, "f16"): (ROWS, 8, False),
         (2, 64, 16, 48, 10240, "f16"): (ROWS, 4, True), (2, 128, 24, 48, 10240, "bf16"): (ROWS, 4, True),
         (2, 32, 32, 48, 3584, "f16"): (ROWS, 4, False), (2, 32, 24, 48, 5120, "f16"): (0, 0, False)}


@pytest.mark.parametrize("call", CALLS, ids=lambda c: "w%d-g%d-m%d-%dx%d-%s" % c)
def test_what_the_calls_launch(lutq, call):
    bits, group, M, N, K, dtype = call
    p = lutq.calib_plan(bits, group, M, N, K, 0 if dtype == "f16" else 1)
    assert (p.scheduling, p.row_blocks_per_wave, p.scheduling == ROWS and p.tiles_per_item > 0) == CALLS[call], p


@pytest.mark.gpu
@pytest.mark.parametrize("call", CALLS, ids=lambda c: "w%d-g%d-m%d-%dx%d-%s" % c)
def test_scalar_table_as_a_codebook(lutq, call):
    import torch
    bits, group, M, N, K, dtype = call
    c = gen.make_case(N + M, M, N, K, bits, group, dtype, "random_index")
    d = DeviceCase(lutq, c)
    want = to_bits(d.matmul(lutq))
    rows = np.unique(np.concatenate([np.arange(16), np.arange(N - 16, N), np.random.default_rng(M).choice(N, min(N, 64), replace=False)]))
    check_y(want[:, rows], gen.Case(M, len(rows), K, bits, group, dtype, c.X, c.Q[rows], c.S[rows], c.T), str(call))
    e, dim = np.arange(256), 8 // bits
    book = to_dev(np.stack([c.T[(e >> (bits * j)) & ((1 << bits) - 1)] for j in range(dim)], axis=1), dtype)
    Y = torch.full((M, N), float("nan"), dtype=d.X.dtype, device="cuda")
    (lutq.lutq_matmul_pairs if bits == 4 else lutq.lutq_matmul_quads)(d.X, d.packed, d.S, book, group, Y, d.ws)
    assert np.array_equal(to_bits(Y), want)
    assert not d.ws[:65536].any().item()
