"""A particle's kick and move in given fields do not depend on which kernel pushes it:
a simulation of its own spreads up to 2^16 particles over 4 lanes each, a batch takes
one lane a particle, and momenta and positions after one step are equal bit for bit
(the gathers' fused operations are the same ones in the same order)."""
import numpy as np
import pytest

import pic_inputs as pi
import test_gpu_rows as rows
from paper_1505_04007_amd import native

pytestmark = pytest.mark.gpu

P, W, C = native.BC_PERIODIC, native.BC_PEC, native.BC_CPML


@pytest.mark.parametrize("n,bc", [((20, 9, 7), (W, W, W)), ((20, 9, 7), (P, P, P)), ((19, 12, 11), (C, P, C)),
                                  ((17, 1, 6), (W, P, W)), ((2, 2, 2), (W, P, W)), ((1, 3, 5), (P, W, P)),
                                  ((2, 1, 4), (P, P, P))])
@pytest.mark.parametrize("count", [1, 15, 17, 64, 65, 1000, 1 << 16])
def test_alone_and_batched(n, bc, count):
    rng = np.random.default_rng(count + n[0])
    b = rows._bunch(n, (0, 0, 0), n, count, rng, False)
    E = [3e11 * rng.standard_normal(n) for _ in range(3)]
    H = [3e11 / 376.73 * rng.standard_normal(n) for _ in range(3)]
    z = np.zeros(n)
    got = []
    for batch in (False, True):
        s = native.Simulation(*n, 2e-9, pi.courant_dt(2e-9), z, z, bc=bc, npml=3, bunch=b, init_E=E, init_H=H)
        p0 = s.particles()
        if batch:
            native.Batch([s]).step(1)
        else:
            s.step(1)
        got.append(s.particles())
        assert not np.array_equal(got[-1][3:], p0[3:])
    assert np.array_equal(got[0], got[1], equal_nan=True)
