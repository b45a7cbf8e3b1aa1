"""PFMI_SERVER_TWO_STEP=0: one step per batched launch, deep tiles included (the
launch counter counts the launches of each captured tick)."""
import numpy as np
import pytest

import paper_2511_10508_amd as P
from test_gpu_serving import _alone, _serve

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ndim,shape", [(2, (1, 200, 300)), (3, (30, 47, 52))])
def test_one_step_per_launch(monkeypatch, ndim, shape):
    monkeypatch.setenv("PFMI_SERVER_TWO_STEP", "0")
    monkeypatch.setenv("PFMI_SERVER_TUNE", "off")
    r = dict(id=0, kind=P.PF_AC, ndim=ndim, shape=shape, steps=64, order=2, params=[1.0, 1.0], dt=0.03, seed=5,
             arrival=0.0, fp32=True, cube_side=3)
    results, st = _serve([r], steps_per_tick=16)
    assert st["captures"] > 0 and st["launches"] == st["captures"] * 16, st
    res, fields = results[0]
    assert res["status"] == 0 and np.array_equal(_alone(r)[0][0], fields[0])


def test_a_row_of_two_million_sites_marches(monkeypatch):
    """Two steps per launch, not eight: deep tiles would compute 64 rows to write one."""
    monkeypatch.setenv("PFMI_SERVER_TUNE", "off")
    r = dict(id=0, kind=P.PF_AC, ndim=2, shape=(1, 1, 2000000), steps=32, order=2, params=[1.0, 1.0], dt=0.03, seed=5,
             arrival=0.0, fp32=True, cube_side=3)
    results, st = _serve([r], steps_per_tick=16)
    assert st["captures"] > 0 and st["launches"] == st["captures"] * 16 // 2, st
    res, fields = results[0]
    assert res["status"] == 0 and np.array_equal(_alone(r)[0][0], fields[0])
