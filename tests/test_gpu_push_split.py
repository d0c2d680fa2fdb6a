"""The push of few particles (4 lanes a particle) against the general one, which a
batch always runs: the same bunch in a simulation of its own and in a batch of one.

Currents: the one-step cases of test_gpu_rows, and dense bunches on either side
of the largest number of particles that is spread.  An edge sums at most some
700 FP32 terms, in another order on either side: 700^(1/2) roundings of 2^-25
at most each, 8e-7 of it, so 5e-6 of the field's norm.  Kicks: a gathered value
is 8 products summed in FP32, some 10 roundings of at most 2^-24 of the largest
field on either side, and a kick here is no more than the momentum: 2e-6 of the
largest momentum."""
import numpy as np
import pytest

import pic_inputs as pi
import test_gpu_rows as rows
from paper_1505_04007_amd import native

pytestmark = pytest.mark.gpu

CASES = [m.args[1] for m in rows.test_one_step_current.pytestmark if m.name == "parametrize" and "," in m.args[0]][0]
SPLIT_MAX = 1 << 16


def _sim(n, bc, bunch, mode=0, E=None):
    z = np.zeros(n)
    return native.Simulation(*n, 2e-9, pi.courant_dt(2e-9), z, z, bc=bc, npml=3, bunch=bunch, deposit_mode=mode,
                             init_E=E)


def _one_step(n, bc, bunch, batch, mode=0, E=None):
    s = _sim(n, bc, bunch, mode, E)
    if batch:
        native.Batch([s]).step(1)
    else:
        s.step(1)
    return s.fields(native.FIELD_E), s.particles()


@pytest.mark.parametrize("cold", [True, False])
@pytest.mark.parametrize("n,bc,lo,hi,count", CASES)
def test_same_current_as_the_general_push(n, bc, lo, hi, count, cold):
    b = rows._bunch(n, lo, hi, count, np.random.default_rng(count), cold)
    E0, _ = _one_step(n, bc, b, False)
    E1, _ = _one_step(n, bc, b, True)
    assert np.linalg.norm(E1) > 0
    assert np.linalg.norm(E0 - E1) <= 5e-6 * np.linalg.norm(E1)


@pytest.mark.parametrize("count", [SPLIT_MAX - 1, SPLIT_MAX, SPLIT_MAX + 1])
@pytest.mark.parametrize("lo,hi", [((4, 2, 2), (44, 10, 10)), ((6, 5, 5), (30, 8, 8))])
def test_dense_bunch(count, lo, hi):
    n, bc = (48, 12, 12), (native.BC_PEC,) * 3
    b = rows._bunch(n, lo, hi, count, np.random.default_rng(count), False)
    E0, _ = _one_step(n, bc, b, False)
    E1, _ = _one_step(n, bc, b, False, mode=1)
    assert np.linalg.norm(E0 - E1) <= 5e-6 * np.linalg.norm(E1)


@pytest.mark.parametrize("n,bc", [((20, 9, 7), (rows.W, rows.W, rows.W)), ((20, 9, 7), (rows.P, rows.P, rows.P)),
                                  ((17, 1, 6), (rows.W, rows.P, rows.W)), ((2, 2, 2), (rows.W, rows.P, rows.W)),
                                  ((1, 3, 5), (rows.P, rows.W, rows.P))])
@pytest.mark.parametrize("count", [1, 15, 64, 65, 1000])
def test_same_kick_as_the_general_push(n, bc, count):
    rng = np.random.default_rng(count)
    b = rows._bunch(n, (0, 0, 0), n, count, rng, False)
    E = [3e11 * rng.standard_normal(n) for _ in range(3)]
    _, p0 = _one_step(n, bc, b, False, E=E)
    _, p1 = _one_step(n, bc, b, True, E=E)
    assert np.array_equal(np.isnan(p0), np.isnan(p1))
    for k in range(6):
        scale = np.nanmax(np.abs(p1[3:])) if k > 2 else max(n) * 2e-9
        assert np.nanmax(np.abs(p0[k] - p1[k]), initial=0.0) <= 2e-6 * scale
