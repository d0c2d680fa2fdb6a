"""Field kernels over runs of 256 cells in memory order (the whole grid's, and a
band of 16 rows'): rows shorter and longer than a run, one-cell axes, ragged
last runs and bands.  The cells' arithmetic is that of the 64 x 4 tile, so E, H
and J_pol are equal bit for bit, also after the adjoint's runs (same gradient)."""
import numpy as np
import pytest

import pic_inputs as pi
from paper_1505_04007_amd import native

pytestmark = pytest.mark.gpu

P, W, C = native.BC_PERIODIC, native.BC_PEC, native.BC_CPML


@pytest.mark.parametrize("n,bc", [
    ((1, 1, 1), (P, P, P)),
    ((2, 2, 2), (W, W, W)),
    ((3, 1, 400), (W, P, C)),
    ((300, 1, 9), (C, P, W)),
    ((255, 5, 3), (P, W, P)),
    ((256, 17, 3), (W, C, P)),
    ((257, 16, 4), (C, C, W)),
    ((130, 33, 5), (C, P, W)),
    ((700, 3, 2), (P, P, W)),
    ((19, 48, 8), (W, C, W)),
])
def test_runs_equal_tiles(n, bc):
    rng = np.random.default_rng(sum(n))
    dx = 2e-9
    wp = np.where(rng.random(n) < 0.3, pi.AG_WP, 0.0)
    E = [rng.standard_normal(n) for _ in range(3)]
    got = []
    for shape in (0, 3, 11, None):
        s = native.Simulation(*n, dx, pi.courant_dt(dx), wp, 0.01 * wp, bc=bc, npml=3 if C in bc else 0, init_E=E)
        if shape is not None:
            s.tune(force=shape)
        s.step(7)
        got.append([s.fields(f) for f in (native.FIELD_E, native.FIELD_H, native.FIELD_JPOL)])
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert np.array_equal(a, b)
