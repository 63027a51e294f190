"""lutq_quantize where its table of cells decides least: weights on and beside every decision threshold, tables that are
not ascending, hold equal, nearly equal or very large entries, and scales that are zero, subnormal, near the ends of the type or infinite.
Indices and scales equal the oracle's (fp64 division and scan) bit for bit."""
import numpy as np
import pytest

import lutq_inputs as gen
from gpu_util import to_bits, to_dev, torch_dtype
from oracle import lutq_oracle as orc

pytestmark = pytest.mark.gpu


def tables(bits, dtype, rng):
    E = 1 << bits
    asc = np.sort(rng.standard_normal(E))
    asc /= np.abs(asc).max()
    yield "symmetric", np.linspace(-1, 1, E)                       # a threshold at exactly zero
    yield "learned", asc
    yield "descending", asc[::-1]
    yield "shuffled", rng.permutation(asc)
    yield "duplicates", np.sort(rng.choice(asc, E))
    yield "crowded", np.sort(np.concatenate([[-1.0], 0.3 + rng.standard_normal(E - 2) * 1e-3, [1.0]]))   # many thresholds per cell
    yield "beyond one", asc * 1.7                                  # thresholds at magnitudes above 1
    yield "large", np.concatenate([asc[:-1], [30000.0]])           # distances whose rounding could reorder them
    if dtype == "bf16":                                            # different entries that fp64 distances cannot tell apart
        yield "nearly equal", np.concatenate([[1e-30, -1e-25, 3e-20], asc[3:]])


@pytest.mark.parametrize("bits", (2, 3, 4))
@pytest.mark.parametrize("dtype", ("f16", "bf16"))
def test_quantize_thresholds_tables_and_scales(lutq, bits, dtype):
    import torch
    rng = np.random.default_rng(bits)
    N, K = 64, 1024
    for ti, (name, T64) in enumerate(tables(bits, dtype, rng)):
        group = (32, 64, 128, 256)[ti % 4]
        T = gen.encode16(np.asarray(T64), dtype)
        t = np.unique(orc.to_f64(T, dtype))
        W = (rng.standard_normal((N, K)) * 0.02).astype(np.float32)
        # a scale of exactly 1, and weights at the thresholds, one fp32 step and some 1e-6 to 1e-4 beside them
        mids = ((t[:-1] + t[1:]) / 2) if len(t) > 1 else np.zeros(1)
        mids = mids[np.abs(mids) < 1]
        if len(mids):
            off = rng.choice([0, 0, 1e-7, -1e-7, 2e-6, -2e-6, 8e-6, -8e-6, 3e-5, -3e-5, 1e-4, -1e-4], (16, K))
            W[:16] = np.clip(rng.choice(mids, (16, K)) + off, -1, 1).astype(np.float32)
            W[1] = np.nextafter(W[1], np.float32(2))
            W[:16, ::32] = 1.0
        W[16] = 0.0
        W[17] *= np.float32(2.0 ** -14)                             # fp16: subnormal scales, or zero ones
        W[18] *= np.float32(2.0 ** -22)
        W[19] *= np.float32(2.0 ** -126)                            # bf16: the smallest scales
        W[20] *= np.float32(2.0 ** 20)                              # fp16: an infinite scale
        W[21] *= np.float32(2.0 ** 120)                             # bf16: the largest ones
        W[22] = (2.0 ** rng.integers(-30, 1, K) * rng.choice([-1.0, 1.0], K)).astype(np.float32)
        for w16 in (False, True):
            if w16:
                with np.errstate(over="ignore"):
                    Wb = gen.encode16(W, dtype)
                W64 = orc.to_f64(Wb, dtype)
                W64[~np.isfinite(W64)] = 0.0                        # (weights are finite)
                Wd = to_dev(gen.encode16(W64, dtype), dtype)
            else:
                W64, Wd = W.astype(np.float64), torch.from_numpy(W).cuda()
            with np.errstate(over="ignore"):
                Q, S = orc.quantize(W64, T, group, dtype)
            # a scale of zero makes u = 0 against every entry: the nearest to zero, the lowest of equal ones
            S_out = torch.zeros((N, K // group), dtype=torch_dtype(dtype), device="cuda")
            P_out = torch.zeros(lutq.lutq_packed_bytes(N, K, bits, group), dtype=torch.uint8, device="cuda")
            lutq.lutq_quantize(Wd, to_dev(T, dtype), bits, group, S_out, P_out)
            what = f"b{bits} {dtype} g{group} {name} w16={w16}"
            assert np.array_equal(to_bits(S_out), S), what
            got = lutq.lutq_unpack(P_out.cpu().numpy(), N, K, bits, group)
            bad = np.argwhere(got != Q)
            assert not len(bad), f"{what}: {len(bad)} indices differ, first at {bad[0]}"


def test_quantize_more_units_than_wavefronts(lutq):
    """Every wavefront walks several units, the last stride runs past the end: 4112 x 4096 and a single row block."""
    import torch
    rng = np.random.default_rng(9)
    T = gen.encode16(gen.normal_float_table(4), "f16")
    for N, K, group in ((4112, 4096, 256), (16, 128, 32), (16, 65536, 128)):
        W = rng.standard_normal((N, K)).astype(np.float32)
        S_out = torch.zeros((N, K // group), dtype=torch.float16, device="cuda")
        P_out = torch.zeros(N * K // 2, dtype=torch.uint8, device="cuda")
        lutq.lutq_quantize(torch.from_numpy(W).cuda(), to_dev(T, "f16"), 4, group, S_out, P_out)
        got = lutq.lutq_unpack(P_out.cpu().numpy(), N, K, 4, group)
        rows = np.unique(np.concatenate([np.arange(min(N, 16)), np.arange(N - 16, N), rng.choice(N, 32)]))
        Q, S = orc.quantize(W[rows].astype(np.float64), T, group, "f16")
        assert np.array_equal(got[rows], Q) and np.array_equal(to_bits(S_out)[rows], S), (N, K, group)


@pytest.mark.parametrize("bits", (2, 3, 4))
@pytest.mark.parametrize("dtype", ("f16", "bf16"))
@pytest.mark.parametrize("w16", (False, True))
def test_quantize_weights_that_are_not_finite(lutq, bits, dtype, w16):
    """Weights are to be finite; one that is not spoils its own group and nothing else, and looks nothing up outside the table of
    cells (whose addresses are formed from the weights)."""
    import torch
    rng = np.random.default_rng(20 + bits)
    N, K, group = 48, 2048, 32 if w16 else 64
    T = gen.encode16(gen.normal_float_table(bits), dtype)
    W = (rng.standard_normal((N, K)) * 0.02).astype(np.float32)
    clean = np.ones((N, K // group), dtype=bool)
    for r, v in ((0, np.inf), (1, -np.inf), (2, np.nan), (17, np.inf), (18, -np.nan), (40, np.nan)):
        c = rng.integers(0, K, 5)
        W[r, c] = v
        clean[r, c // group] = False
    if not w16:
        W[3, 100:102] = np.array([0x7fffffff, 0xffffffff], dtype=np.uint32).view(np.float32)      # rounds past the last NaN to a zero
        clean[3, 100 // group] = False
    Wt = torch.from_numpy(W).cuda()
    Wd = Wt.to(torch_dtype(dtype)) if w16 else Wt
    W64 = np.where(np.isfinite(W), Wd.double().cpu().numpy(), 0.0)
    Q, S = orc.quantize(W64, T, group, dtype)
    S_out = torch.zeros((N, K // group), dtype=torch_dtype(dtype), device="cuda")
    P_out = torch.zeros(lutq.lutq_packed_bytes(N, K, bits, group), dtype=torch.uint8, device="cuda")
    lutq.lutq_quantize(Wd, to_dev(T, dtype), bits, group, S_out, P_out)
    got = lutq.lutq_unpack(P_out.cpu().numpy(), N, K, bits, group)
    full = np.repeat(clean, group, axis=1)
    assert np.array_equal(to_bits(S_out)[clean], S[clean])
    assert np.array_equal(got[full], Q[full])


@pytest.mark.parametrize("bits", (2, 3, 4))
@pytest.mark.parametrize("dtype", ("f16", "bf16"))
def test_quantize_beyond_the_cells(lutq, bits, dtype):
    """Whole matrices of the smallest scales, where |u| is up to 1.5 (fp16), of infinite ones and of those beyond 2^-100 and 2^100
    (bf16), and a mixture; tables without an entry below 1000, with entries that cancel, and with thresholds above 1."""
    import torch
    rng = np.random.default_rng(40 + bits)
    N, K, group, E = 32, 1024, 64, 1 << bits
    asc = np.sort(rng.standard_normal(E))
    tables = {"nf": gen.normal_float_table(bits), "far": np.linspace(1100, 2000, E), "opposite": np.linspace(-60000, 60000, E),
              "far shuffled": rng.permutation(np.linspace(-9000, 30000, E)), "wide": asc / np.abs(asc).max() * 1.9, "near": asc * 1e-3}
    tiny = 2.0 ** -24
    matrices = {"least": rng.uniform(-1.49, 1.49, (N, K)) * tiny, "two": rng.uniform(-2.49, 2.49, (N, K)) * tiny,
                "subnormal": rng.standard_normal((N, K)) * 1e-5, "infinite": rng.standard_normal((N, K)) * 1e6,
                "small": rng.standard_normal((N, K)) * 2.0 ** -106, "large": rng.standard_normal((N, K)) * 2.0 ** 106}
    mixed = rng.standard_normal((N, K)) * 0.02
    for i, m in enumerate(matrices.values()):
        mixed[3 * i] = m[0]
        mixed[3 * i + 1, group:2 * group] = m[1, :group]
    matrices["mixed"] = mixed
    for tname, T64 in tables.items():
        T = gen.encode16(np.asarray(T64), dtype)
        for mname, W64 in matrices.items():
            W = W64.astype(np.float32)
            with np.errstate(over="ignore"):
                Q, S = orc.quantize(W.astype(np.float64), T, group, dtype)
            S_out = torch.zeros((N, K // group), dtype=torch_dtype(dtype), device="cuda")
            P_out = torch.zeros(lutq.lutq_packed_bytes(N, K, bits, group), dtype=torch.uint8, device="cuda")
            lutq.lutq_quantize(torch.from_numpy(W).cuda(), to_dev(T, dtype), bits, group, S_out, P_out)
            what = f"b{bits} {dtype} {tname} {mname}"
            assert np.array_equal(to_bits(S_out), S), what
            got = lutq.lutq_unpack(P_out.cpu().numpy(), N, K, bits, group)
            assert np.array_equal(got, Q), f"{what}: {np.count_nonzero(got != Q)} indices differ"
