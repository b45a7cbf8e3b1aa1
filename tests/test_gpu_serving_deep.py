"""Served requests on deep tiles (several steps per batched launch): bitwise the
same request stepped alone, at grids of a tile less or more, requests of one
class with different sizes and different steps left in a tick."""
import numpy as np
import pytest

import paper_2511_10508_amd as P
from test_gpu_serving import _alone, _serve

pytestmark = pytest.mark.gpu

PARAMS = {P.PF_AC: ([1.0, 1.0], 0.03), P.PF_CH: ([1.0, 1.0], 0.004), P.PF_GS: ([0.2, 0.1, 0.04, 0.06], 0.3),
          P.PF_MC: ([1.0, 1.0, 0.5], 0.01)}
# above the grids kept whole in LDS; 64 columns or rows are exactly one tile
SHAPES = {2: [(1, 515, 64), (1, 64, 517), (1, 191, 193), (1, 301, 147)],
          3: [(20, 47, 32), (33, 32, 31), (9, 61, 70), (41, 29, 30)]}


@pytest.mark.parametrize("fp32", [True, False], ids=["fp32", "fp64"])
@pytest.mark.parametrize("order", [2, 4])
@pytest.mark.parametrize("kind", [P.PF_AC, P.PF_CH, P.PF_GS, P.PF_MC], ids=["ac", "ch", "gs", "mc"])
@pytest.mark.parametrize("ndim", [2, 3])
def test_deep_served_requests_are_bitwise_those_stepped_alone(ndim, kind, order, fp32):
    params, dt = PARAMS[kind]
    reqs = [dict(id=i, kind=kind, ndim=ndim, shape=shape, steps=15 + 11 * i, order=order, params=params, dt=dt,
                 seed=300 + i, arrival=0.0, fp32=fp32, cube_side=3) for i, shape in enumerate(SHAPES[ndim])]
    results, _ = _serve(reqs, steps_per_tick=11)
    for r in reqs:
        res, fields = results[r["id"]]
        assert res["status"] == 0 and res["steps_done"] == r["steps"]
        for a, b in zip(_alone(r)[0], fields):
            assert np.array_equal(a, b), r


def test_a_lone_request_takes_eight_steps_per_launch(monkeypatch):
    """Marching tiles take a launch per two steps: the counter, which counts the launches
    of each captured tick, tells the paths apart."""
    monkeypatch.setenv("PFMI_SERVER_TUNE", "off")
    r = dict(id=0, kind=P.PF_AC, ndim=2, shape=(1, 200, 300), steps=64, order=2, params=[1.0, 1.0], dt=0.03, seed=5,
             arrival=0.0, fp32=False, cube_side=3)
    _, st = _serve([r], steps_per_tick=16)
    assert st["captures"] > 0 and st["launches"] == st["captures"] * 16 // 8, st
