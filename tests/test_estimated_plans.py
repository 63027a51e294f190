"""Calls of up to 32 rows without a plan on shapes where the estimated times, not the rules, choose the launch: row streaming in
uneven K slices, with scale rows that are not whole 16-byte units, several passes, and single teams of odd wave counts."""
import numpy as np
import pytest

import lutq_inputs as gen
import paper_2407_10960_amd as lutq
from gpu_util import DeviceCase, to_bits
from test_gpu_parity import check_y

# (bits, group, M, N, K, dtype)
SHAPES = [(4, 256, 22, 1328, 23296, "bf16"), (2, 64, 21, 1136, 13312, "f16"), (3, 32, 20, 2368, 4096, "f16"), (4, 64, 13, 1248, 21504, "bf16"),
          (2, 32, 9, 21904, 1536, "bf16"), (3, 64, 15, 8880, 4352, "bf16"), (4, 256, 12, 12304, 1536, "bf16"), (2, 64, 14, 14256, 3328, "bf16"),
          (4, 256, 17, 26704, 1792, "f16"), (3, 32, 9, 5072, 1536, "bf16"), (4, 64, 11, 10304, 1280, "f16"), (3, 256, 10, 22672, 1536, "bf16"),
          # panels of one block of 32 rows, with and without K slices
          (4, 32, 17, 1072, 22528, "f16"), (2, 32, 25, 2128, 12288, "bf16"), (3, 64, 32, 4272, 8192, "f16"), (4, 64, 27, 9200, 3584, "bf16"),
          (2, 32, 32, 1152, 20992, "f16"), (3, 32, 18, 6000, 5376, "bf16"),
          (4, 128, 6, 4448, 11648, "bf16"), (2, 32, 1, 19056, 1024, "f16"), (4, 32, 2, 11536, 3968, "f16"), (3, 64, 3, 9040, 2560, "bf16")]


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
