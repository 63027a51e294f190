"""lutq_dequant at the edges of its launch: a single tile, fewer tiles than compute units, four and eight wavefronts per
workgroup, few and many workgroups per compute unit, a last stride that runs past the end, super-blocks of one, two and four
row blocks, groups longer than a tile, stores through and past the caches.  Bit for bit the oracle's weights; rows around the matrix stay as they were."""
import numpy as np
import pytest

import lutq_inputs as gen
from gpu_util import DeviceCase, to_bits, torch_dtype
from oracle import lutq_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", (4, 3, 2))
@pytest.mark.parametrize("dtype", ("f16", "bf16"))
def test_dequant_edges(lutq, bits, dtype):
    import torch
    tile = 128 if bits == 4 else 256
    # (row blocks, K tiles, group): 2, 30, 1290, 4100, 6150 (eight wavefronts at 4 bits), 9234 and 12561 tiles (eight workgroups per unit)
    for i, (nb, kt, group) in enumerate([(1, 2, 256), (5, 6, 32), (258, 5, 64), (1025, 4, 128), (1025, 6, 64), (513, 18, 256), (4187, 3, 32)]):
        c = gen.make_case(60 + i, 1, 16 * nb, kt * tile, bits, group, dtype, "random_index")
        d = DeviceCase(lutq, c)
        W = torch.full((c.N + 32, c.K), 7.0, dtype=torch_dtype(dtype), device="cuda")
        lutq.lutq_dequant(d.packed, d.S, d.T, bits, group, W[16:16 + c.N])
        got = to_bits(W[16:16 + c.N])
        want = orc.dequant(c.Q, c.T, c.S, group, dtype)
        assert np.array_equal(got, want), f"b{bits} {dtype} N{c.N} K{c.K} g{group}: {np.count_nonzero(got != want)} differ"
        assert (W[:16] == 7.0).all().item() and (W[16 + c.N:] == 7.0).all().item()


@pytest.mark.parametrize("bits,dtype", ((4, "f16"), (3, "bf16"), (2, "f16"), (4, "bf16")))
def test_dequant_past_the_caches(lutq, bits, dtype):
    """8192 x 8192, the least matrix that is written past the caches, and one row block less: 96 sampled rows bit for bit, and a
    product that reads the matrix right after gives the same as one that reads a copy."""
    import torch
    group, rng = 64, np.random.default_rng(bits)
    for N in (8192, 8176):
        c = gen.make_case(90 + bits, 4, N, 8192, bits, group, dtype, "random_index")
        d = DeviceCase(lutq, c)
        W = torch.full((N, c.K), 7.0, dtype=torch_dtype(dtype), device="cuda")
        lutq.lutq_dequant(d.packed, d.S, d.T, bits, group, W)
        Y = torch.mm(d.X, W.t())
        rows = np.unique(np.concatenate([np.arange(16), np.arange(N - 16, N), rng.choice(N, 64, replace=False)]))
        assert np.array_equal(to_bits(W)[rows], orc.dequant(c.Q[rows], c.T, c.S[rows], group, dtype)), f"b{bits} {dtype} N{N}"
        assert torch.equal(Y, torch.mm(d.X, W.clone().t())) and not (W == 7.0).all(dim=1).any().item()
