"""The fixed-point deposit's matrix-core sums: from one window for a whole wavefront to
one for every lane, wraps, walls and thin grids.  The units are whole numbers and their
sums exact, so J_b does not depend on which particles share a wavefront: the same bunch in
reverse and in shuffled order gives the same current bit for bit.  Against the
floating-point deposit an edge differs by half a unit (2^-25 of a particle's largest
current) per particle and the FP32 sums' rounding: 5e-6 of the field's norm."""
import numpy as np
import pytest

import pic_inputs as pi
import test_gpu_rows as rows
from paper_1505_04007_amd import native

pytestmark = pytest.mark.gpu

CASES = [m.args[1] for m in rows.test_one_step_current.pytestmark if m.name == "parametrize" and "," in m.args[0]][0]


def _E(n, bc, b, mode, order):
    z = np.zeros(n)
    b = pi.Bunch(*[getattr(b, f)[order] for f in ("x", "y", "z", "ux", "uy", "uz")], b.q, b.m, b.w)
    s = native.Simulation(*n, 2e-9, pi.courant_dt(2e-9), z, z, bc=bc, npml=3, bunch=b, deposit_mode=mode)
    s.step(1)
    return s.fields(native.FIELD_E)


@pytest.mark.parametrize("cold", [True, False])
@pytest.mark.parametrize("n,bc,lo,hi,count", CASES + [
    ((24, 12, 12), (rows.W, rows.W, rows.W), (3, 3, 3), (20, 9, 9), 66),      # a window for nearly every lane
    ((24, 12, 12), (rows.P, rows.P, rows.P), (0, 0, 0), (24, 12, 12), 130),   # the same, many at the edges
    ((12, 8, 8), (rows.W, rows.W, rows.W), (5, 4, 4), (6, 5, 5), 5000),       # one window, full sums
])
def test_sums(n, bc, lo, hi, count, cold):
    rng = np.random.default_rng(count + n[0])
    b = rows._bunch(n, lo, hi, count, rng, cold)
    same = np.arange(count)
    E = _E(n, bc, b, 2, same)
    assert np.array_equal(E, _E(n, bc, b, 2, same[::-1]))
    assert np.array_equal(E, _E(n, bc, b, 2, rng.permutation(count)))
    Ef = _E(n, bc, b, 0, same)
    assert np.linalg.norm(Ef) > 0
    assert np.linalg.norm(E - Ef) <= 5e-6 * np.linalg.norm(Ef)
