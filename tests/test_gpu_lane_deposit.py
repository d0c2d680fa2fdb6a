"""Per-lane atomics (deposit_mode 1, and the lanes left over by the row sums): the edges
of a window outside the grid get nothing, on walls, absorbing layers, wraps and grids
thinner than a window; and the push with one lane a particle, row sums and all, which a
batch runs at any number of particles.

E^1 = -J_b from zero fields.  Against the FP64 oracle by the FP32 positions, 1.2e-4 of
the field's norm as for the row sums; against the fixed-point deposit, whose sums are
exact, by a few hundred FP32 terms and a factor's rounding, 5e-6."""
import numpy as np
import pytest

import pic_inputs as pi
import test_gpu_rows as rows
from oracle import pic_oracle as po
from paper_1505_04007_amd import native

pytestmark = pytest.mark.gpu

P, W, C = native.BC_PERIODIC, native.BC_PEC, native.BC_CPML


def _E(n, bc, bunch, mode, batch=False):
    z = np.zeros(n)
    s = native.Simulation(*n, 2e-9, pi.courant_dt(2e-9), z, z, bc=bc, npml=3, bunch=bunch, deposit_mode=mode)
    if batch:
        native.Batch([s]).step(1)
    else:
        s.step(1)
    return s.fields(native.FIELD_E)


@pytest.mark.parametrize("cold", [True, False])
@pytest.mark.parametrize("n,bc,lo,hi,count", [
    ((48, 12, 12), (W, W, W), (10, 5, 5), (12, 7, 7), 65),
    ((48, 12, 12), (W, W, W), (0, 0, 0), (48, 1, 1), 300),       # along a wall corner
    ((48, 12, 12), (W, W, W), (46, 10, 10), (48, 12, 12), 300),  # into the far corner
    ((48, 12, 12), (C, P, W), (0, 0, 0), (48, 12, 12), 500),
    ((17, 5, 4), (P, P, P), (0, 0, 0), (17, 5, 4), 500),
    ((5, 3, 2), (P, P, P), (0, 0, 0), (5, 3, 2), 300),
    ((40, 1, 9), (W, P, W), (3, 0, 0), (37, 1, 9), 400),
    ((1, 1, 12), (P, P, W), (0, 0, 0), (1, 1, 12), 200),
    ((2, 2, 2), (W, W, W), (0, 0, 0), (2, 2, 2), 150),
])
def test_edges_of_the_grid(n, bc, lo, hi, count, cold):
    b = rows._bunch(n, lo, hi, count, np.random.default_rng(count + cold), cold)
    o = po.OracleSim(*n, 2e-9, pi.courant_dt(2e-9), bc=bc, npml=3, wp_map=np.zeros(n), gamma_map=np.zeros(n))
    o.set_particles(b.x, b.y, b.z, b.ux, b.uy, b.uz, b.q, b.m, b.w)
    o.step(1)
    Eo = np.stack([o.E[c][:n[0], :n[1], :n[2]] for c in range(3)])
    norm = np.linalg.norm(Eo)
    assert norm > 0
    Ex = _E(n, bc, b, 2)
    for E in (_E(n, bc, b, 1), _E(n, bc, b, 1, True), _E(n, bc, b, 0, True)):
        assert np.linalg.norm(E - Eo) <= 1.2e-4 * norm
        assert np.linalg.norm(E - Ex) <= 5e-6 * norm
