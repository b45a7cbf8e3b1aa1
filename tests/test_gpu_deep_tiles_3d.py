"""3D deep-tile kernels (bricks in registers, one or more steps per launch), the
path of 3D models whose tile the caller left to the library: bitwise the per-site
kernels, reductions of every step against exact sums; and the finalising launches
of many steps at once of the marching kernels."""
import math

import numpy as np
import pytest

import synth
import paper_2511_10508_amd as P

pytestmark = pytest.mark.gpu

BASE = {P.PF_AC: ([1.0, 1.0], 0.03), P.PF_CH: ([1.0, 1.0], 0.004), P.PF_GS: ([0.2, 0.1, 0.04, 0.06], 0.3),
        P.PF_MC: ([1.0, 1.0, 0.5], 0.01)}

# thinner than the halo, exactly a brick wide (32) or high (8, 12, .. 32 rows),
# one more and less, several ragged bricks, one plane
SHAPES = [(3, 5, 2), (32, 8, 9), (32, 32, 32), (31, 33, 12), (65, 24, 7), (40, 13, 1), (70, 41, 29)]
STEPS = [1, 2, 7, 12]


def _state(kind, n, seed):
    shape = (n[2], n[1], n[0])
    if kind == P.PF_GS:
        return synth.initial_fields(3, shape, seed, synth.IC_GS_CUBES, (4, 5, 0.01))
    return synth.initial_fields(kind, shape, seed, synth.IC_UNIFORM, (-0.1, 0.1))


def _run(kind, n, order, prec, steps, flags, f0, pin=None):
    params, dt = BASE[kind]
    m = P.Model(P.make_desc(kind, n, dt=dt, order=order, precision=prec, params=params, flags=flags))
    if pin:
        m.set_tile(pin)
    for f, a in enumerate(f0):
        m.set_field(f, a)
    for k in steps:
        m.step(k)
    return [m.get_field(f) for f in range(len(f0))], m


@pytest.mark.parametrize("prec", [P.PF_FP64, P.PF_FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("order", [2, 4])
@pytest.mark.parametrize("kind", [P.PF_AC, P.PF_CH, P.PF_GS, P.PF_MC], ids=["ac", "ch", "gs", "mc"])
def test_deep_bricks_bitwise_the_per_site_kernels(kind, order, prec):
    for i, n in enumerate(SHAPES):
        steps = STEPS[i % len(STEPS)]
        f0 = _state(kind, n, 40 + i)
        ref, _ = _run(kind, n, order, prec, [steps], P.PF_FORCE_GENERIC, f0)
        for flags in (0, P.PF_REDUCE_EACH_STEP):
            got, _ = _run(kind, n, order, prec, [steps], flags, f0)
            for x, y in zip(got, ref):
                assert np.array_equal(x, y), (n, steps, flags)
        got, _ = _run(kind, n, order, prec, [steps // 3, steps - steps // 3], 0, f0)
        for x, y in zip(got, ref):
            assert np.array_equal(x, y), (n, steps)


@pytest.mark.parametrize("prec", [P.PF_FP64, P.PF_FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("order", [2, 4])
@pytest.mark.parametrize("kind", [P.PF_AC, P.PF_CH, P.PF_GS, P.PF_MC], ids=["ac", "ch", "gs", "mc"])
def test_deep_brick_reductions_of_every_step(kind, order, prec):
    """As in 2D: mass to 1e-15 sum|x| of the exact sums of the states, energy and the
    second mass to 1e-13 per site of the marching kernels'; NaN sites counted."""
    steps = 5
    for n in [(5, 7, 3), (34, 40, 21)]:
        f0 = _state(kind, n, 9)
        _, m = _run(kind, n, order, prec, [steps], P.PF_REDUCE_EACH_STEP, f0)
        _, o = _run(kind, n, order, prec, [steps], P.PF_REDUCE_EACH_STEP, f0, pin=4)
        hi, lo = m.reduce_history(P.PF_RED_MASS0, steps)
        _, one = _run(kind, n, order, prec, [], 0, f0)
        for k in range(steps):
            s = one.get_field(0).ravel()
            assert abs(math.fsum([hi[k], lo[k]]) - math.fsum(s)) <= 1e-15 * max(1.0, float(np.abs(s).sum())), (n, k)
            one.step(1)
        second = P.PF_RED_MASS1 if kind in (P.PF_GS, P.PF_MC) else P.PF_RED_ENERGY
        a, b = m.reduce_history(second, steps), o.reduce_history(second, steps)
        assert np.max(np.abs((a[0] + a[1]) - (b[0] + b[1]))) <= 1e-13 * n[0] * n[1] * n[2]
    f0[0][2, 3, 4] = np.nan
    _, m = _run(kind, n, order, prec, [2], P.PF_REDUCE_EACH_STEP, f0)
    _, o = _run(kind, n, order, prec, [2], P.PF_REDUCE_EACH_STEP, f0, pin=4)
    bad, want = m.reduce_history(P.PF_RED_NONFINITE, 2)[0], o.reduce_history(P.PF_RED_NONFINITE, 2)[0]
    assert bad[0] == 1 and np.array_equal(bad, want)


@pytest.mark.parametrize("graph", [0, P.PF_USE_GRAPH], ids=["eager", "graph"])
@pytest.mark.parametrize("tb", [1, 2])
def test_marching_history_is_that_of_single_calls(tb, graph):
    """The reductions of a long call (finalised many steps at a time, some in graphs
    replayed three times with eager calls between) are bitwise those of the same
    steps taken one call per launch."""
    n, kind = (200, 90), P.PF_CH
    f0 = _state(kind, n + (1,), 3)
    hist = []
    for calls in ([70, 5, 101], [tb] * 0):
        params, dt = BASE[kind]
        m = P.Model(P.make_desc(kind, n, dt=dt, order=4, params=params, flags=P.PF_REDUCE_EACH_STEP | graph))
        m.set_tile(16)
        m.set_time_block(tb)
        m.set_field(0, f0[0])
        rows = []
        for c in calls or [k for part in (70, 5, 101) for k in [tb] * (part // tb) + [1] * (part % tb)]:
            m.step(c)
            rows.append(np.stack([np.stack(m.reduce_history(q, c)) for q in (P.PF_RED_MASS0, P.PF_RED_ENERGY)]))
        hist.append(np.concatenate(rows, axis=2))
    assert np.array_equal(hist[0], hist[1])
