"""Device memory of models with per-step reductions: what pf_footprint_bytes
says, and the same however a run is split into calls."""
import pytest
import torch

import paper_2511_10508_amd as P

pytestmark = pytest.mark.gpu

PARAMS = {P.PF_AC: ([1.0, 1.0], 0.02), P.PF_CH: ([1.0, 1.0], 0.004), P.PF_GS: ([0.2, 0.1, 0.04, 0.06], 0.3)}


def _free():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def _model(kind, n, order, prec):
    params, dt = PARAMS[kind]
    m = P.Model(P.make_desc(kind, n, dt=dt, order=order, precision=prec, params=params,
                            flags=P.PF_REDUCE_EACH_STEP))
    m.init(P.PF_IC_UNIFORM, 7, (-0.1, 0.1))
    return m


@pytest.mark.parametrize("kind,n,order,prec", [(P.PF_CH, (128, 128), 2, P.PF_FP64), (P.PF_CH, (256, 256), 4, P.PF_FP32),
                                               (P.PF_GS, (1024, 1024), 2, P.PF_FP64), (P.PF_AC, (96, 96, 96), 2, P.PF_FP32),
                                               (P.PF_CH, (300, 200), 6, P.PF_FP64)])
def test_memory_of_a_reducing_model(kind, n, order, prec):
    _model(kind, n, order, prec).step(2)  # code objects and pools of the runtime
    before = _free()
    m = _model(kind, n, order, prec)
    m.step(1)
    m.reduce(P.PF_RED_MASS0)
    held = before - _free()
    # the history (48 bytes a step, 1024 steps at first) and the allocator's granularity,
    # 2 MiB for each of the model's allocations
    allocations = 2 * m.desc.nfields + 6
    assert held <= P.footprint_bytes(m.desc) + 48 * 1024 + allocations * (2 << 20)
    for steps in (1000, 2, 3, 7, 25, 1):
        m.step(steps)
        assert before - _free() == held, steps


def test_a_history_too_long_for_memory_leaves_a_usable_model():
    m = _model(P.PF_CH, (70, 50), 2, P.PF_FP64)
    m.step(3)
    with pytest.raises(P.PfError):
        m.step(10 ** 10)  # 480 GB of history: refused before anything is launched
    assert m.steps_done() == 3
    m.step(5)
    assert m.steps_done() == 8
    hi, _ = m.reduce_history(P.PF_RED_MASS0, 5)
    assert abs(hi[4] - m.reduce(P.PF_RED_MASS0)[0]) <= 1e-12 * 70 * 50
