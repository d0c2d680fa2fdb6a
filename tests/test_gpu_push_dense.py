"""Dense bunches moving every way: a wavefront holds one wide grid row and the few lanes
beside it that moved back over a cell's face, which are passes of their own there; on
either side of the numbers where that begins and where the push changes its kernel, in
one cell, a few and many, at walls, wraps and on thin grids.

E^1 = -J_b from zero fields, against the fixed-point deposit, whose sums are exact.  An
edge's N terms have random signs, so its sum and its partial sums are of the size of
N^(1/2) terms, and N FP32 additions are off by N^(1/2) 2^-25 of that; a factor's rounding
of 2^-24 is 10 times that of a current of a tenth of a cell: 2^-23 (count^(1/2) + 20) of
the field's norm."""
import numpy as np
import pytest

import pic_inputs as pi
import test_gpu_rows as rows
from paper_1505_04007_amd import native

pytestmark = pytest.mark.gpu

P, W, C = native.BC_PERIODIC, native.BC_PEC, native.BC_CPML


def _E(n, bc, bunch, mode, steps, batch=False):
    z = np.zeros(n)
    s = native.Simulation(*n, 2e-9, pi.courant_dt(2e-9), z, z, bc=bc, npml=3, bunch=bunch, deposit_mode=mode)
    if batch:
        native.Batch([s]).step(steps)
    else:
        s.step(steps)
    return s.fields(native.FIELD_E)


@pytest.mark.parametrize("count", [33, 64, 4096, 4097, 20000, 1 << 16, (1 << 16) + 1])
@pytest.mark.parametrize("n,bc,lo,hi", [
    ((24, 12, 12), (W, W, W), (11, 5, 5), (12, 6, 6)),      # one cell
    ((24, 12, 12), (W, W, W), (4, 5, 5), (20, 7, 7)),       # four rows
    ((24, 12, 12), (P, P, P), (0, 0, 0), (24, 2, 2)),       # the same over every wrap
    ((24, 12, 12), (C, W, W), (20, 10, 10), (24, 12, 12)),  # into the far corner
    ((9, 1, 6), (P, P, W), (0, 0, 0), (9, 1, 2)),
    ((1, 2, 3), (P, P, P), (0, 0, 0), (1, 2, 3)),
])
def test_current_of_a_dense_bunch(n, bc, lo, hi, count):
    b = rows._bunch(n, lo, hi, count, np.random.default_rng(count), False)
    E2 = _E(n, bc, b, 2, 1)
    norm = np.linalg.norm(E2)
    tol = 2.0 ** -23 * (count ** 0.5 + 20)
    assert norm > 0
    assert np.linalg.norm(_E(n, bc, b, 0, 1) - E2) <= tol * norm
    if count <= 4097:  # the general kernel, which is a batch's at any number
        assert np.linalg.norm(_E(n, bc, b, 0, 1, batch=True) - E2) <= tol * norm
