"""2D deep-tile kernels (several steps per launch on register tiles), the path
of models whose tile the caller left to the library: bitwise the per-site
kernels, per-step reductions against exact sums of the same states."""
import math

import numpy as np
import pytest

import synth
import paper_2511_10508_amd as P

pytestmark = pytest.mark.gpu

BASE = {P.PF_AC: ([1.0, 1.0], 0.05), P.PF_CH: ([1.0, 1.0], 0.008), P.PF_GS: ([0.2, 0.1, 0.04, 0.06], 0.4),
        P.PF_MC: ([1.0, 1.0, 0.5], 0.01)}

# grids: smaller than a tile and than its halo, one column or row, exactly a
# tile wide or high (64, 128, 256 columns: periodic by itself), one more and
# one less, several ragged tiles in both directions
SHAPES = [(1, 1), (3, 70), (5, 7), (64, 64), (64, 128), (128, 32), (65, 129), (63, 127), (256, 64), (300, 21),
          (517, 203)]
STEPS = [1, 2, 7, 25]


def _state(kind, n, seed):
    shape = (1, n[1], n[0])
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
    out = [m.get_field(f) for f in range(len(f0))]
    assert m.steps_done() == sum(steps)
    return out, m


@pytest.mark.parametrize("prec", [P.PF_FP64, P.PF_FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("order", [2, 4])
@pytest.mark.parametrize("kind", [P.PF_AC, P.PF_CH, P.PF_GS, P.PF_MC], ids=["ac", "ch", "gs", "mc"])
def test_deep_tiles_bitwise_the_per_site_kernels(kind, order, prec):
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
def test_deep_tile_reductions_of_every_step(kind, order, prec):
    """Mass of every step: correctly rounded sums (math.fsum) of the states,
    stepped one by one, to 1e-15 sum|x|; energy: against the marching kernels'
    (other partition) to 1e-13 sum|e|, the repository's bound for both.  NaN
    sites are counted exactly."""
    steps = 9
    for n in [(5, 7), (64, 64), (130, 77), (300, 210)]:
        f0 = _state(kind, n, 9)
        _, m = _run(kind, n, order, prec, [steps], P.PF_REDUCE_EACH_STEP, f0)
        _, o = _run(kind, n, order, prec, [steps], P.PF_REDUCE_EACH_STEP, f0, pin=8)
        hi, lo = m.reduce_history(P.PF_RED_MASS0, steps)
        _, one = _run(kind, n, order, prec, [], 0, f0)
        for k in range(steps):
            s = one.get_field(0).ravel()
            assert abs(math.fsum([hi[k], lo[k]]) - math.fsum(s)) <= 1e-15 * max(1.0, float(np.abs(s).sum())), (n, k)
            one.step(1)
        second = P.PF_RED_MASS1 if kind in (P.PF_GS, P.PF_MC) else P.PF_RED_ENERGY
        a, b = m.reduce_history(second, steps), o.reduce_history(second, steps)
        scale = n[0] * n[1]  # |e| and |x| are of order one at most
        assert np.max(np.abs((a[0] + a[1]) - (b[0] + b[1]))) <= 1e-13 * scale
        assert np.all(m.reduce_history(P.PF_RED_NONFINITE, steps)[0] == 0)
    f0[0][0, 3, 4] = np.nan
    _, m = _run(kind, n, order, prec, [2], P.PF_REDUCE_EACH_STEP, f0)
    _, o = _run(kind, n, order, prec, [2], P.PF_REDUCE_EACH_STEP, f0, pin=8)
    bad, want = m.reduce_history(P.PF_RED_NONFINITE, 2)[0], o.reduce_history(P.PF_RED_NONFINITE, 2)[0]
    assert bad[0] == 1 and np.array_equal(bad, want)
