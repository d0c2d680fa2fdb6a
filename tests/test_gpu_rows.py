"""The row deposit (matrix-core sums of a grid row's particles) where it can go
wrong: rows narrower, as wide and wider than its 16 x nodes, wavefronts of one,
few and many rows, ragged wavefronts, walls and wraps, and grids thinner than
a window.

From zero fields in vacuum one step leaves E^1 = -J_b (times dt / eps0) and
nothing else, so E shows every deposited value.  Tolerances: against per-lane
atomics (deposit_mode 1, same positions and factors) an edge's sum differs by
the rounding of at most a few hundred FP32 terms, 5e-6 of the field's norm.
Against the FP64 oracle, by the FP32 positions: half an ulp of a coordinate
below 64 cells is 1.9e-6, against a move of 0.1 cells or more that a current is
proportional to, 2e-5 per end of a move and axis, six in all: 1.2e-4.
"""
import numpy as np
import pytest

import pic_inputs as pi
from oracle import pic_oracle as po
from paper_1505_04007_amd import native

pytestmark = pytest.mark.gpu

P, W, C = native.BC_PERIODIC, native.BC_PEC, native.BC_CPML


def _bunch(n, lo, hi, count, rng, cold):
    """count particles uniform over cells [lo, hi) moving 0.1 to 0.2 cells a step, along +x or every way."""
    dx = 2e-9
    pos = [rng.uniform(lo[a], hi[a], count) * dx for a in range(3)]
    v = rng.uniform(0.4, 0.7, count)
    d = np.zeros((3, count))
    d[0] = 1.0
    if not cold:
        d = rng.standard_normal((3, count))
        d = np.sign(d) * (0.5 + np.abs(d))
        d /= np.linalg.norm(d, axis=0)
    u = d * v / np.sqrt(1 - v * v) * pi.C_LIGHT
    return pi.Bunch(*pos, *u, -pi.E_CHARGE, pi.M_E, 100.0)


def _E(n, bc, bunch, mode):
    z = np.zeros(n)
    s = native.Simulation(*n, 2e-9, pi.courant_dt(2e-9), z, z, bc=bc, npml=3, bunch=bunch, deposit_mode=mode)
    s.step(1)
    return s.fields(native.FIELD_E)


@pytest.mark.parametrize("cold", [True, False])
@pytest.mark.parametrize("n,bc,lo,hi,count", [
    ((48, 12, 12), (W, W, W), (8, 6, 6), (9, 7, 7), 64),         # one window
    ((48, 12, 12), (W, W, W), (8, 6, 6), (22, 7, 7), 130),       # a row of 14 bases, two wavefronts and 2 lanes
    ((48, 12, 12), (W, W, W), (8, 6, 6), (23, 7, 7), 64),        # 15 bases: one more than a pass takes
    ((48, 12, 12), (W, W, W), (2, 6, 6), (45, 7, 7), 200),       # several passes along one row
    ((48, 12, 12), (W, W, W), (4, 4, 4), (40, 8, 8), 64),        # many rows with few lanes each
    ((48, 12, 12), (W, W, W), (10, 5, 5), (12, 7, 7), 1),
    ((48, 12, 12), (W, W, W), (10, 5, 5), (12, 7, 7), 2),
    ((48, 12, 12), (W, W, W), (10, 5, 5), (14, 7, 7), 700),      # a few rows in every wavefront
    ((48, 12, 12), (W, W, W), (0, 0, 0), (48, 1, 1), 900),       # along a wall corner
    ((48, 12, 12), (C, W, W), (40, 10, 10), (48, 12, 12), 900),  # into the far corner
    ((48, 12, 12), (P, P, P), (0, 0, 0), (48, 12, 12), 900),     # wraps on every axis
    ((17, 5, 4), (P, P, P), (0, 0, 0), (17, 5, 4), 500),
    ((16, 4, 4), (W, P, P), (0, 0, 0), (16, 4, 4), 500),
    ((5, 3, 2), (P, P, P), (0, 0, 0), (5, 3, 2), 300),           # narrower than the pass's nodes
    ((40, 1, 9), (W, P, W), (3, 0, 2), (37, 1, 7), 600),         # one cell across the beam
    ((1, 1, 12), (P, P, W), (0, 0, 2), (1, 1, 10), 200),
    ((2, 2, 2), (W, W, W), (0, 0, 0), (2, 2, 2), 150),
])
def test_one_step_current(n, bc, lo, hi, count, cold):
    rng = np.random.default_rng(count + 7 * n[0] + cold)
    b = _bunch(n, lo, hi, count, rng, cold)
    E0, E1 = _E(n, bc, b, 0), _E(n, bc, b, 1)
    o = po.OracleSim(*n, 2e-9, pi.courant_dt(2e-9), bc=bc, npml=3, wp_map=np.zeros(n), gamma_map=np.zeros(n))
    o.set_particles(b.x, b.y, b.z, b.ux, b.uy, b.uz, b.q, b.m, b.w)
    o.step(1)
    Eo = np.stack([o.E[c][:n[0], :n[1], :n[2]] for c in range(3)])
    norm = np.linalg.norm(Eo)
    assert norm > 0
    assert np.linalg.norm(E0 - E1) <= 5e-6 * norm
    assert np.linalg.norm(E0 - Eo) <= 1.2e-4 * norm
