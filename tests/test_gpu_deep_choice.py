"""Which kernels a model steps on (the launches per step of pf_timing_read): deep
tiles take more of them than the time block of the marching kernels."""
import numpy as np
import pytest

import paper_2511_10508_amd as P

pytestmark = pytest.mark.gpu

STEPS = 24


def _model(kind, n, order=2, prec=P.PF_FP32, flags=0):
    params, dt = {P.PF_AC: ([1.0, 1.0], 0.02), P.PF_CH: ([1.0, 1.0], 0.004),
                  P.PF_GS: ([0.2, 0.1, 0.04, 0.06], 0.3), P.PF_MC: ([1.0, 1.0, 0.5], 0.01)}[kind]
    m = P.Model(P.make_desc(kind, n, dt=dt, order=order, precision=prec, params=params, flags=flags))
    m.init(P.PF_IC_UNIFORM, 7, (-0.1, 0.1))
    return m


def _deep(m, steps=STEPS):
    """Whether a call of `steps` steps ran on deep tiles."""
    m.timing(True)
    m.step(steps)
    _, launches, done = m.timing_read()
    m.timing(False)
    assert done == steps
    return launches < -(-steps // m.time_block())


def test_a_chosen_layout_or_pass_count_is_taken():
    m = _model(P.PF_GS, (40, 30, 20))
    assert _deep(m)
    m.set_tile_rows(2)
    assert not _deep(m)
    m.set_tile_rows(0)
    assert _deep(m)
    m = _model(P.PF_CH, (40, 30, 20))
    assert _deep(m)
    m.set_passes(2)
    assert m.passes() == 2 and not _deep(m)
    m.set_passes(1)
    assert m.passes() == 1 and not _deep(m)


def test_a_chosen_tile_is_taken_until_the_choice_is_given_back():
    m = _model(P.PF_CH, (200, 150))
    assert _deep(m)
    m.set_passes(1)  # no choice in 2D
    assert _deep(m)
    m.set_tile(16)
    assert not _deep(m)
    m.set_tile(0)
    assert _deep(m)
    m.set_time_block(1)
    assert not _deep(m)
    m.set_tile(0)  # the time block stays
    assert not _deep(m)


@pytest.mark.parametrize("kind,n,order,prec", [(P.PF_CH, (1024, 1024), 4, P.PF_FP64),
                                               (P.PF_GS, (96, 96, 96), 2, P.PF_FP32)])
def test_autotuned_models_with_reductions_stay_on_deep_tiles_where_faster(kind, n, order, prec):
    """Deep tiles take half the marching kernels' time or less at these sizes: the
    tuned model keeps them, and so does a later model of its class."""
    red = P.PF_REDUCE_EACH_STEP
    m = _model(kind, n, order, prec, red)
    assert _deep(m)
    before = [m.get_field(f) for f in range(m.desc.nfields)]
    m.autotune(2)
    for f, a in enumerate(before):
        assert np.array_equal(m.get_field(f), a)
    assert m.tile()[0] == 0 and m.time_block() == 1 and m.tile_rows() == 0
    assert _deep(m)
    m.set_tile(16)
    assert m.tile()[0] == 16 and not _deep(m)
    assert _deep(_model(kind, n, order, prec, red))
    # the history of a tuned model: as in the marching kernels' partition
    a, b = _model(kind, n, order, prec, red), _model(kind, n, order, prec, red)
    b.set_tile(16)
    for x in (a, b):
        x.step(STEPS)
    u, v = a.reduce_history(P.PF_RED_MASS0, STEPS), b.reduce_history(P.PF_RED_MASS0, STEPS)
    assert np.max(np.abs((u[0] + u[1]) - (v[0] + v[1]))) <= 1e-15 * a.nsites


@pytest.mark.parametrize("kind,n,order,prec", [(P.PF_GS, (1800, 1800), 4, P.PF_FP64),
                                               (P.PF_MC, (4096, 4096), 4, P.PF_FP64)])
def test_autotuner_times_steps_that_alternate_buffers(kind, n, order, prec):
    """Deep tiles take three quarters of the marching kernels' time here (11 against 15
    us a step, 53 against 62); timed on one unchanging input buffer the marching kernels
    came out ahead.  The state is untouched."""
    m = _model(kind, n, order, prec)
    before = [m.get_field(f) for f in range(m.desc.nfields)]
    m.autotune()
    for f, a in enumerate(before):
        assert np.array_equal(m.get_field(f), a)
    assert m.tile()[0] == 0 and _deep(m)


def test_a_call_of_one_step_marches_where_that_is_faster():
    """Two FP64 fields with reductions, 1024^2: the sums of a call of one step have the
    partition of the marching kernels, bitwise, those of a call of two have not."""
    n, red = (1024, 1000), P.PF_REDUCE_EACH_STEP
    a, b = _model(P.PF_GS, n, 2, P.PF_FP64, red), _model(P.PF_GS, n, 2, P.PF_FP64, red)
    b.set_time_block(1)
    same = {}
    for steps in (1, 2):
        for m in (a, b):
            m.step(steps)
        same[steps] = all(np.array_equal(x, y) for q in (P.PF_RED_MASS0, P.PF_RED_MASS1)
                          for x, y in zip(a.reduce_history(q, steps), b.reduce_history(q, steps)))
    assert same == {1: True, 2: False}
    assert np.array_equal(a.get_field(0), b.get_field(0)) and np.array_equal(a.get_field(1), b.get_field(1))


def test_thin_grids_march_where_tiles_are_mostly_halo():
    """Grids of a few rows or planes, wide enough to fill the chip: a tile computes tens
    of rows to write them.  Small thin grids stay on deep tiles, where the launch counts."""
    for kind, n, order, prec in ((P.PF_GS, (400000, 1), 2, P.PF_FP32), (P.PF_CH, (400000, 2), 4, P.PF_FP64),
                                 (P.PF_MC, (2000000, 4), 4, P.PF_FP32), (P.PF_CH, (1, 500, 500), 4, P.PF_FP64)):
        for flags in (0, P.PF_REDUCE_EACH_STEP):
            assert not _deep(_model(kind, n, order, prec, flags)), (n, flags)
    for kind, n in ((P.PF_GS, (5000, 1)), (P.PF_AC, (1, 5000)), (P.PF_GS, (60, 60, 1)), (P.PF_MC, (700, 500))):
        assert _deep(_model(kind, n)), n


def test_tuned_deep_models_with_reductions_have_the_defaults_partition():
    """A reducing model that the autotuner put on deep tiles, whatever tile it had before:
    every call's sums are bitwise those of a model with the library's choices."""
    n, red = (700, 500), P.PF_REDUCE_EACH_STEP
    ref = _model(P.PF_GS, n, 2, P.PF_FP64, red)
    m = _model(P.PF_GS, n, 2, P.PF_FP64, red)
    m.set_tile(24)
    m.autotune(2)
    assert m.tile()[0] == 0
    for steps in (1, 2, 9):
        for x in (ref, m):
            x.step(steps)
        for q in (P.PF_RED_MASS0, P.PF_RED_MASS1):
            for a, b in zip(ref.reduce_history(q, steps), m.reduce_history(q, steps)):
                assert np.array_equal(a, b), steps
