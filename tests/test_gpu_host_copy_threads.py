"""Host transfers of one model from several threads: fields, a window and a
field being set, of different sizes, all exact."""
import threading

import numpy as np
import pytest

import paper_2511_10508_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [P.PF_FP64, P.PF_FP32], ids=["fp64", "fp32"])
def test_transfers_of_one_model_from_several_threads(prec):
    m = P.Model(P.make_desc(P.PF_MH, (1030, 700), dt=0.001, precision=prec))
    rng = np.random.default_rng(11)
    want = [rng.standard_normal(m.shape).astype(np.float32).astype(np.float64) for _ in range(3)]
    m.set_field(0, want[0])
    m.set_field(1, want[1])
    ref = {"f0": want[0], "f1": want[1], "w": want[1][:, 5:25, 3:43]}
    calls = {"f0": lambda: m.get_field(0), "f1": lambda: m.get_field(1),
             "w": lambda: m.get_window(1, (0, 5, 3), (1, 20, 40))}
    wrong = []

    def read(key):
        for rep in range(20):
            if not np.array_equal(calls[key](), ref[key]):
                wrong.append((key, rep))

    def write():
        for _ in range(20):
            m.set_field(2, want[2])

    threads = [threading.Thread(target=read, args=(k,)) for k in calls] + [threading.Thread(target=write)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong, wrong
    assert np.array_equal(m.get_field(2), want[2])
