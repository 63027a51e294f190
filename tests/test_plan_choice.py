"""What a call of 1..32 rows launches, asked of the host logic (no device): a plan means itself, whoever gives it; only a call without
one, or with the empty one, takes the library's choice."""
import numpy as np
import pytest

import lutq_inputs as gen
from gpu_util import DeviceCase, to_bits
from test_gpu_parity import check_y


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


def test_a_call_without_a_plan_fits_the_built_in_scratch(lutq):
    """Also where neither the rules' plan nor the one for little scratch does (the first three)."""
    ws = lutq.STATIC_SCRATCH_BYTES
    refused = [(2, 256, 31, 45408, 26624, 0, 256), (2, 32, 31, 18720, 7168, 1, 256), (4, 32, 24, 64480, 16896, 0, 256)]
    for p in refused:
        with pytest.raises(lutq.LutqError) as e:
            lutq.calib_plan(*p, ws, plan=lutq.lutq_plan_default_for(*p))
        assert e.value.code == 11
    # (the last of these: only a plan of few partial sums fits)
    for p in refused + [(4, 64, 32, 57344, 8192, 1, 256)] + list(problems(7, 3000)):
        plan = lutq.calib_plan(*p, ws)
        assert plan == lutq.Plan() or plan.grid > 0
        assert lutq.calib_plan(*p, ws, plan=lutq.Plan()) == plan, p


def test_a_remembered_choice_is_that_of_its_problem(lutq):
    """The choice is kept for the last problems: more of them than there is room for, twice over, at two scratch sizes."""
    first = {}
    for turn in range(2):
        for p in problems(6, 1500):
            for ws in (None, lutq.STATIC_SCRATCH_BYTES):
                assert first.setdefault((p, ws), (lutq.calib_plan(*p, ws), lutq.calib_route(*p, ws))) == \
                    (lutq.calib_plan(*p, ws), lutq.calib_route(*p, ws)), p


# panels of 32 rows are the library's choice on these: (bits, group, M, N, K, dtype)
PANELS = [(4, 32, 17, 1072, 22528, 0), (3, 64, 32, 4272, 8192, 0), (2, 32, 32, 1152, 20992, 0)]
IMPOSSIBLE = ((1, 0, 8, 2, 3), (1, 256, 16, 2, 1, 2, 4), (0, 0, 0, 0, 0, 7))   # waves that are no three teams, a queue, no scheduling


@pytest.mark.parametrize("p", PANELS)
def test_a_registered_plan_keeps_a_call_off_the_panels_only_if_it_runs(lutq, p):
    bits, group, M, N, K, dt = p

    def registered(plan, m_max=32):
        try:
            lutq.lutq_plan_table_set([(bits, group, dt, 1, m_max, N, K, plan)])
            return lutq.calib_plan(*p)
        finally:
            lutq.lutq_plan_table_set([])

    assert lutq.calib_plan(*p) == lutq.Plan()
    rules = lutq.lutq_plan_default_for(*p)
    assert registered(rules) == rules
    assert registered(rules, 16) == lutq.Plan() and registered(lutq.Plan()) == lutq.Plan()
    for plan in IMPOSSIBLE:
        assert lutq.lutq_plan_check(*p, 256, lutq.Plan(*plan)) == 10
        assert registered(lutq.Plan(*plan)) == lutq.Plan(), plan


@pytest.mark.gpu
@pytest.mark.parametrize("p", PANELS)
def test_registered_plans_give_the_bits_of_the_same_plan_passed(lutq, p):
    bits, group, M, N, K, dt = p
    c = gen.make_case(N + M, M, N, K, bits, group, "bf16" if dt else "f16", "random_index")
    d = DeviceCase(lutq, c)
    free = to_bits(d.matmul(lutq))
    check_y(free, c, str(p))
    rules = lutq.lutq_plan_default(*p)
    given = to_bits(d.matmul(lutq, plan=rules))
    check_y(given, c, f"{p} {rules}")
    for plan, want in [(rules, given), (lutq.Plan(), free)] + [(lutq.Plan(*q), free) for q in IMPOSSIBLE]:
        try:
            lutq.lutq_plan_table_set([(bits, group, dt, 1, 32, N, K, plan)])
            assert np.array_equal(to_bits(d.matmul(lutq)), want), plan
        finally:
            lutq.lutq_plan_table_set([])
    assert not np.array_equal(free, given)           # (two orders of summation)


# (bits, group, M, N, K, dtype): panels; row streaming in K slices; the rules' plan
TUNED = [((2, 32, 23, 4272, 22272, 0), "panels"), ((4, 64, 13, 1248, 21504, 1), "estimated"), ((4, 128, 8, 4096, 4096, 0), "rules")]


@pytest.mark.gpu
@pytest.mark.parametrize("p,what", TUNED)
def test_tuner_times_the_call_without_a_plan_and_the_rules(lutq, p, what):
    """Each launch is timed once; the tuner's result, registered, leaves a call with the launch that was timed."""
    import torch
    bits, group, M, N, K, dt = p
    c = gen.make_case(N + M, M, N, K, bits, group, "bf16" if dt else "f16", "random_index")
    d = DeviceCase(lutq, c)
    rules, free = lutq.lutq_plan_default(*p), lutq.calib_plan(*p)
    assert what == ("panels" if free == lutq.Plan() else "rules" if free == rules else "estimated")
    cands = lutq.lutq_tune_candidates(*p)
    assert cands[:2] == [lutq.Plan(), rules] if what != "rules" else cands[0] == rules and lutq.Plan() not in cands
    assert len(set(map(repr, cands))) == len(cands) and (what != "estimated" or free not in cands)
    Y = torch.empty((M, N), dtype=d.X.dtype, device="cuda")
    best, us = lutq.lutq_tune(d.X, [d.packed, d.packed.clone()], [d.S, d.S.clone()], d.T, bits, group, Y, d.ws, reps=2)
    assert us > 0.5 and best in cands
    want = to_bits(d.matmul(lutq, plan=best))
    check_y(want, c, f"{p} {best}")
    try:
        lutq.lutq_plan_table_set([(bits, group, dt, 1, 32, N, K, best)])
        assert np.array_equal(to_bits(d.matmul(lutq)), want)
    finally:
        lutq.lutq_plan_table_set([])
    assert not d.ws[:65536].any().item()


# (bits, group, M, N, K, dtype), us of the rules' launch, us of another that estimates have preferred or prefer: pairs a tenth apart
MEASURED = [((3, 32, 6, 880, 20480, 0), 10.3, 15.1), ((3, 32, 5, 1216, 16384, 0), 9.8, 13.9), ((3, 32, 15, 512, 13824, 1), 10.0, 13.9),
            ((2, 32, 10, 512, 16384, 0), 10.5, 12.9), ((3, 32, 10, 41056, 2048, 0), 16.5, 20.5), ((3, 32, 24, 688, 5632, 0), 10.5, 12.5),
            ((3, 32, 26, 800, 5632, 1), 10.9, 13.1), ((3, 32, 24, 608, 4608, 1), 10.1, 11.9),
            ((3, 64, 16, 12464, 1280, 0), 8.6, 12.7), ((3, 64, 16, 13232, 1280, 1), 9.4, 13.6), ((2, 64, 14, 28720, 1280, 1), 17.9, 20.7),
            ((3, 128, 8, 42448, 2048, 1), 15.6, 17.8), ((4, 128, 13, 4224, 1664, 1), 5.6, 6.4), ((3, 64, 14, 16032, 2304, 1), 9.8, 11.2),
            ((2, 64, 15, 25328, 2048, 0), 18.4, 10.0), ((4, 256, 23, 5232, 4864, 0), 18.1, 10.7), ((3, 128, 30, 30704, 1280, 0), 25.6, 11.2),
            ((4, 256, 24, 1104, 16384, 0), 18.9, 11.6), ((3, 256, 32, 6704, 4864, 0), 22.3, 12.0), ((2, 256, 10, 30512, 3328, 0), 25.9, 12.9),
            ((4, 32, 21, 1888, 16768, 0), 25.8, 13.9), ((3, 64, 12, 4464, 15104, 1), 29.0, 18.1), ((2, 128, 8, 20784, 11264, 0), 39.9, 23.9)]


def test_a_call_without_a_plan_takes_the_faster_launch(lutq):
    """Cold weights, 256 compute units."""
    for p, rules_us, other_us in MEASURED:
        assert (lutq.calib_plan(*p) == lutq.lutq_plan_default_for(*p)) == (rules_us < other_us), p
