"""Graph replay of the marching kernels without reductions: models with a chosen
tile take them (deep tiles are launched directly), bitwise the eager launches, over
several calls with eager work between the replays."""
import numpy as np
import pytest

import paper_2511_10508_amd as P
from test_gpu_parity import BASE, dt_for, fields_for

pytestmark = pytest.mark.gpu


def _model(kind, ndim, shape, order, prec, flags, f0):
    params = BASE[kind][0]
    n = (shape[2], shape[1], shape[0])[:ndim]
    m = P.Model(P.make_desc(kind, n, dt=dt_for(kind, ndim, order, params), order=order, precision=prec, params=params,
                            flags=flags))
    m.set_tile(16)
    for f, a in enumerate(f0):
        m.set_field(f, a)
    return m


@pytest.mark.parametrize("prec", [P.PF_FP64, P.PF_FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("order", [2, 4])
@pytest.mark.parametrize("ndim,shape", [(2, (1, 67, 277)), (3, (19, 35, 70))])
@pytest.mark.parametrize("kind", [P.PF_AC, P.PF_CH, P.PF_GS, P.PF_MC], ids=["ac", "ch", "gs", "mc"])
def test_graph_replay_of_marching_kernels_is_bitwise_eager(kind, ndim, shape, order, prec):
    f0 = fields_for(kind, shape, 19)
    a = _model(kind, ndim, shape, order, prec, 0, f0)
    b = _model(kind, ndim, shape, order, prec, P.PF_USE_GRAPH, f0)
    for steps in (70, 3, 129, 64):  # graphs of 32 steps from 64 steps a call on
        for m in (a, b):
            m.step(steps)
        for f in range(len(f0)):
            assert np.array_equal(a.get_field(f), b.get_field(f)), steps
        assert a.reduce(P.PF_RED_MASS0) == b.reduce(P.PF_RED_MASS0)
    # the path they took: a launch per step
    a.timing(True)
    a.step(64)
    assert a.timing_read()[1] == 64


@pytest.mark.parametrize("kind,ndim,shape,order", [(P.PF_CH, 2, (1, 40, 70), 10), (P.PF_CH, 3, (11, 20, 30), 8),
                                                   (P.PF_MC, 2, (1, 40, 70), 12)])
def test_graph_replay_of_per_site_kernels_is_bitwise_eager(kind, ndim, shape, order):
    """Orders that run the per-site kernels, which hold a field-sized temporary: it is there
    before the first capture."""
    params = BASE[kind][0]
    n = (shape[2], shape[1], shape[0])[:ndim]
    dt = 0.5 * dt_for(kind, ndim, order, params)
    f0 = fields_for(kind, shape, 23)
    got = []
    for flags in (0, P.PF_USE_GRAPH):
        m = P.Model(P.make_desc(kind, n, dt=dt, order=order, params=params, flags=flags))
        assert m.tile()[1] == 1
        for f, a in enumerate(f0):
            m.set_field(f, a)
        for steps in (64, 5, 70):
            m.step(steps)
        got.append([m.get_field(f) for f in range(len(f0))])
    for x, y in zip(*got):
        assert np.array_equal(x, y)
