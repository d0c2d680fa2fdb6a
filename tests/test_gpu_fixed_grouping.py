"""The fixed-point deposit's sums do not depend on which particles share a wavefront.

pic_init puts every bunch in one order, so the same bunch with some particles before it
is what changes the grouping: ones that leave through the wall in their first step
deposit nothing and only shift the rest by so many lanes, and carry a bunch over 2^16
particles, where scattered wavefronts change from lane by lane to the matrix cores.
Without walls they deposit in planes that the bunch does not reach.  Units are whole
numbers and their sums exact: E^1 = -J_b is equal bit for bit."""
import numpy as np
import pytest

import pic_inputs as pi
import test_gpu_rows as rows
from paper_1505_04007_amd import native

pytestmark = pytest.mark.gpu

P, W, C = native.BC_PERIODIC, native.BC_PEC, native.BC_CPML
F = ("x", "y", "z", "ux", "uy", "uz")
LEAST = 1 << 16


def _join(a, b):
    return pi.Bunch(*[np.concatenate([getattr(a, f), getattr(b, f)]) for f in F], a.q, a.m, a.w)


def _E(n, bc, bunch):
    z = np.zeros(n)
    s = native.Simulation(*n, 2e-9, pi.courant_dt(2e-9), z, z, bc=bc, npml=3, bunch=bunch, deposit_mode=2)
    s.step(1)
    return s.fields(native.FIELD_E)


def _leaving(k):
    """k particles in the first cell, out through x = 0 in one step."""
    u = -10.0 * pi.C_LIGHT
    return pi.Bunch(np.full(k, 0.01 * 2e-9), np.full(k, 1e-9), np.full(k, 1e-9), np.full(k, u), np.zeros(k), np.zeros(k),
                    -pi.E_CHARGE, pi.M_E, 100.0)


@pytest.mark.parametrize("cold", [True, False])
@pytest.mark.parametrize("n,bc,lo,hi,count", [
    ((24, 12, 12), (W, W, W), (5, 4, 4), (6, 5, 5), 700),        # one cell: up to 8 windows
    ((24, 12, 12), (W, W, W), (3, 3, 3), (7, 5, 5), 300),        # 16 cells: around one product's windows
    ((24, 12, 12), (W, W, W), (3, 3, 3), (20, 9, 9), 400),       # a window for nearly every lane
    ((24, 12, 12), (C, P, P), (0, 0, 0), (24, 12, 12), 900),     # walls and wraps
    ((20, 1, 9), (W, P, W), (0, 0, 0), (20, 1, 9), 500),
    ((2, 2, 2), (W, W, W), (0, 0, 0), (2, 2, 2), 150),
])
def test_shifted_by_lanes(n, bc, lo, hi, count, cold):
    b = rows._bunch(n, lo, hi, count, np.random.default_rng(count + cold), cold)
    E = _E(n, bc, b)
    assert np.abs(E).max() > 0
    for k in (1, 7, 31, 63):
        assert np.array_equal(E, _E(n, bc, _join(_leaving(k), b))), k


@pytest.mark.parametrize("count", [2000, 40000])
def test_over_the_largest_number_taken_lane_by_lane(count):
    n, bc = (48, 40, 40), (W, W, W)  # 2000: every window a lane's own
    b = rows._bunch(n, (0, 0, 0), n, count, np.random.default_rng(count), False)
    E = _E(n, bc, b)
    for more in (LEAST - count, LEAST - count + 1):
        assert np.array_equal(E, _E(n, bc, _join(_leaving(more), b))), more


@pytest.mark.parametrize("cold", [True, False])
@pytest.mark.parametrize("count", [100, 600])
def test_every_axis_wraps(count, cold):
    n, bc = (20, 9, 12), (P, P, P)
    rng = np.random.default_rng(count)
    b = rows._bunch(n, (0, 0, 7), (20, 9, 12), count, rng, cold)  # nodes 6 .. 11, 0, 1 along z
    E = _E(n, bc, b)
    planes = [0, 1, 6, 7, 8, 9, 10, 11]
    assert np.abs(E).max() > 0 and not E[:, :, :, 2:6].any()
    for k in (1, 7, 31, 63):
        more = rows._bunch(n, (0, 0, 3), (20, 9, 4), k, rng, cold)  # nodes 2 .. 5
        assert np.array_equal(E[..., planes], _E(n, bc, _join(more, b))[..., planes]), k
