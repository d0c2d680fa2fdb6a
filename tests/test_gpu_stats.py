"""The live particles and pushes of stats(), against the particles read back: a
step pushes those that are still live after it.  Whole numbers, no tolerance."""
import numpy as np
import pytest

import pic_inputs as pi
from paper_1505_04007_amd import native

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("count", [1, 63, 65, 1023, 1024, 1025, 70000, 262145])  # to more than one sweep of the grid
def test_counts(count, mode):
    n, dx = (24, 10, 9), 2e-9
    rng = np.random.default_rng(count)
    pos = [rng.uniform(0, n[d], count) * dx for d in range(3)]
    u = 1.5e8 * rng.standard_normal((3, count))
    b = pi.Bunch(*pos, *u, -pi.E_CHARGE, pi.M_E, 1e-6)
    z = np.zeros(n)
    s = native.Simulation(*n, dx, pi.courant_dt(dx), z, z, bc=(0, 1, 0), npml=3, bunch=b, deposit_mode=mode)
    pushes = 0
    for _ in range(3):
        s.step(1)
        live = int(np.sum(~np.isnan(s.particles()[0])))
        pushes += live
        st = s.stats()
        assert (st["live"], st["pushes"], st["steps"]) == (live, pushes, _ + 1)
    cells = np.floor(np.array(pos) / dx).astype(int)
    assert st["pbox"] == tuple(cells.min(1)) + tuple(cells.max(1))
    assert s.diag()["count"] == live
