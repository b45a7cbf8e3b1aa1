"""Spectral step on power-of-two grids, whose transforms are the library's own:
every length of both kernels (rows 64..8192, columns 32..4096), 2D and 3D, both
models and precisions, against the numpy oracle after a few steps, with a state set
from outside between them.

Tolerance: a transform of N values errs by at most a few eps log2 N of the largest
spectrum value relative to the field's norm; over 6 steps, each amplifying by at most
1.06, 1e-13 (FP64) and 5e-6 (FP32) of max|u| = 0.1 are over ten times that."""
import numpy as np
import pytest

from oracle import spectral
import synth
import paper_2511_10508_amd as P

pytestmark = pytest.mark.gpu

GRIDS = [(64, 32), (64, 4096), (128, 64), (256, 128), (512, 256), (1024, 512), (2048, 1024), (4096, 2048), (8192, 32),
         (64, 32, 32), (128, 64, 256), (64, 128, 64)]


@pytest.mark.parametrize("prec", [P.PF_FP64, P.PF_FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("n", GRIDS, ids=["x".join(map(str, g)) for g in GRIDS])
def test_own_transforms_against_numpy(n, prec):
    kind = P.PF_CH if (n[0] + n[1]) % 3 else P.PF_AC
    ndim = len(n)
    shape = tuple(reversed(tuple(n) + (1,) * (3 - ndim)))
    f0 = synth.initial_fields(kind, shape, 41, synth.IC_UNIFORM, (-0.1, 0.1))[0]
    params, dx, dt = [1.0, 1.0], 0.9, 0.2
    ref = spectral.run(kind, f0, ndim, dx, dt, params, 6)
    d = P.make_desc(kind, n, dx=dx, dt=dt, order=2, precision=prec, params=params, flags=P.PF_SPECTRAL)
    m = P.Model(d)
    m.set_field(0, f0)
    m.step(2)
    m.set_field(0, m.get_field(0))  # the kept spectrum is dropped: the state is transformed again
    m.step(4)
    err = float(np.max(np.abs(m.get_field(0) - ref)))
    assert err <= (1e-14 if prec == P.PF_FP64 else 5e-7), err
