"""Host transfers through the pinned halves (4 MiB each): fields that fill a
part of one, several, and rows longer than one, with and without row padding;
windows against numpy indexing.  All exact."""
import numpy as np
import pytest

import paper_2511_10508_amd as P

pytestmark = pytest.mark.gpu

GRIDS = [(1,), (7, 3), (515, 389), (1024, 1024), (1023, 1700), (524287, 2), (1048577, 3), (1200001,), (33, 129, 65)]


@pytest.mark.parametrize("prec", [P.PF_FP64, P.PF_FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("n", GRIDS, ids=["x".join(map(str, n)) for n in GRIDS])
def test_set_get_and_window_exact(n, prec):
    d = P.make_desc(P.PF_GS, n, dt=0.1, precision=prec)
    m = P.Model(d)
    shape = m.shape
    rng = np.random.default_rng(5)
    want = []
    for f in range(2):
        a = rng.standard_normal(shape)
        m.set_field(f, a)
        want.append(a.astype(np.float32).astype(np.float64) if prec == P.PF_FP32 else a)
    for f in range(2):
        assert np.array_equal(m.get_field(f), want[f])
    for origin, w in (((0, 0, 0), shape), ((-1, -2, -3), tuple(max(1, s // 2) for s in shape)),
                      ((shape[0] - 1, shape[1] - 1, shape[2] - 1), tuple(min(s, 5) for s in shape))):
        got = m.get_window(1, origin, w)
        ix = np.ix_(*[(np.arange(k) + o) % s for k, o, s in zip(w, origin, shape)])
        assert np.array_equal(got, want[1][ix])
