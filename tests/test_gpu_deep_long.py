"""A column too long for one launch of deep tiles (2^32 threads): the model marches."""
import numpy as np
import pytest

import paper_2511_10508_amd as P

pytestmark = pytest.mark.gpu


def test_a_column_of_2_29_sites_steps():
    def model(ny):
        m = P.Model(P.make_desc(P.PF_AC, (1, ny), dt=0.05, order=2, precision=P.PF_FP32, params=[1.0, 1.0]))
        m.init(P.PF_IC_CONST, 0, (0.25,))
        m.step(24)
        return m

    want = model(300).get_field(0)[0, 0, 0]
    m = model(1 << 29)
    for y in (0, (1 << 29) - 1, 123456789):
        assert np.all(m.get_window(0, (0, y, 0), (1, 7, 1)) == want), y
