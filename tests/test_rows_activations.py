"""Row streaming of 17..32 rows: activations loaded in operand order (fewer rows) and turned into operands through LDS (more rows)
are two instances of one kernel.  A row's sum does not depend on the rows beside it, so both give a row the same bits."""
import numpy as np
import pytest

import lutq_inputs as gen
from gpu_util import DeviceCase, to_bits, to_dev
from test_gpu_parity import check_y, tk


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("bits,side", [(4, 4), (4, 8), (3, 4), (2, 4), (2, 8)])
@pytest.mark.parametrize("slices", [1, 3])
def test_rows_do_not_depend_on_how_activations_are_loaded(bits, side, dtype, slices):
    import paper_2407_10960_amd as lutq
    nb, kt, group = (11, 7, 64) if slices == 1 else (13, 20, 32)
    c = gen.make_case(31 * bits + side, 32, 16 * nb, tk(bits) * kt, bits, group, dtype, "random_index")
    d = DeviceCase(lutq, c)
    plan = lutq.Plan(side, 2, 0, 2, nb // 2, 3) if slices == 1 else lutq.Plan(side, 3 * -(-nb // side), 0, 2, nb // -(-nb // side), 3, 7)
    all_rows = to_bits(d.matmul(lutq, plan=plan))
    check_y(all_rows, c, f"b{bits} {dtype} {plan}")
    for M in range(17, 32):
        assert np.array_equal(to_bits(d.matmul(lutq, plan=plan, X=d.X[:M].contiguous())), all_rows[:M]), M
    assert not d.ws[:65536].any().item()


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("bits,nb", [(4, 515), (4, 1285), (3, 515), (3, 1285), (2, 515), (4, 40), (3, 40), (2, 40)])
def test_the_same_with_one_table_per_row(bits, nb, dtype):
    import torch
    import paper_2407_10960_amd as lutq
    K, group = (512, 64) if nb > 100 else (8192, 64)
    c = gen.make_case(nb, 32, 16 * nb, K, bits, group, dtype, "random_index")
    d = DeviceCase(lutq, c)
    T = to_dev(gen.encode16(np.random.default_rng(nb).standard_normal((c.N, 1 << bits)), dtype), dtype)

    def run(M):
        Y = torch.full((M, c.N), float("nan"), dtype=d.X.dtype, device="cuda")
        lutq.lutq_matmul_channel(d.X[:M].contiguous(), d.packed, d.S, T, bits, group, Y, d.ws)
        return to_bits(Y)
    turned = run(32)
    assert np.array_equal(run(25)[:23], turned[:23])
    few = run(20)
    assert np.array_equal(run(17), few[:17])
    assert np.array_equal(few, turned[:20])
