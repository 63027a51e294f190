"""What a call of 1..32 rows launches, asked of the host logic (no device): a plan means itself, whoever gives it; only a call without
one, or with the empty one, takes the library's choice."""
import numpy as np
import pytest


def problems(seed, count, m_min=1):
    """(bits, group, M, N, K, dtype, compute units)"""
    rng = np.random.default_rng(seed)
    while count:
        bits, group = int(rng.choice([2, 3, 4])), int(rng.choice([32, 64, 128, 256]))
        step = max(group, 128 if bits == 4 else 256)
        K = step * int(np.exp(rng.uniform(0, np.log(32768 / step))))
        N = 16 * int(np.exp(rng.uniform(0, np.log(6000))))
        M, dt, cus = int(rng.integers(m_min, 33)), int(rng.integers(0, 2)), int(rng.choice([256, 256, 256, 304, 64]))
        if N * K * bits // 8 < 1 << 31:
            count -= 1
            yield bits, group, M, N, K, dt, cus


@pytest.mark.parametrize("small_scratch", [False, True])
def test_a_given_plan_is_what_runs(lutq, small_scratch):
    """The rules' plan, passed back, runs -- also where a call without a plan takes another launch -- and so does that other one."""
    ws = lutq.STATIC_SCRATCH_BYTES if small_scratch else None
    others = panels = 0
    for p in problems(5, 1500):
        rules = lutq.lutq_plan_default_for(*p)
        try:
            runs = lutq.calib_plan(*p, ws, plan=rules)
        except lutq.LutqError as e:
            assert small_scratch and e.code == 11, (p, rules)      # its partial sums do not fit
            continue
        assert runs == rules, p
        free = lutq.calib_plan(*p, ws)
        assert lutq.calib_plan(*p, ws, plan=lutq.Plan()) == free, p
        if free == lutq.Plan():
            panels += 1
        else:
            assert lutq.calib_plan(*p, ws, plan=free) == free, p
            others += free != rules
    assert others > 100 and panels > 50
