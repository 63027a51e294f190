"""lutq_dequant at the edges of its launch: a single tile, fewer tiles than compute units, 4 to 16 wavefronts per
workgroup, a last stride that runs past the end, super-blocks of one, two and four row blocks, groups longer than a
tile.  Bit for bit the oracle's weights; rows around the matrix stay as they were."""
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
    # (row blocks, K tiles, group): 1, 30, 1290 (six wavefronts), 4100 (sixteen, just over one round), 9234 tiles
    for i, (nb, kt, group) in enumerate([(1, 2, 256), (5, 6, 32), (258, 5, 64), (1025, 4, 128), (513, 18, 256)]):
        c = gen.make_case(60 + i, 1, 16 * nb, kt * tile, bits, group, dtype, "random_index")
        d = DeviceCase(lutq, c)
        W = torch.full((c.N + 32, c.K), 7.0, dtype=torch_dtype(dtype), device="cuda")
        lutq.lutq_dequant(d.packed, d.S, d.T, bits, group, W[16:16 + c.N])
        got = to_bits(W[16:16 + c.N])
        want = orc.dequant(c.Q, c.T, c.S, group, dtype)
        assert np.array_equal(got, want), f"b{bits} {dtype} N{c.N} K{c.K} g{group}: {np.count_nonzero(got != want)} differ"
        assert (W[:16] == 7.0).all().item() and (W[16 + c.N:] == 7.0).all().item()
