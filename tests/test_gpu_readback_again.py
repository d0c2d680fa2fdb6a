"""Arrays read back before, at and after the pinned staging comes in: at 256 KB of one
array on either side, and small ones from the ninth on.  Values are moved, not
computed: every read gives the FP32 state."""
import numpy as np
import pytest

import pic_inputs as pi
from paper_1505_04007_amd import native

pytestmark = pytest.mark.gpu

DX = 2e-9


def _sim(n, count, **kw):
    rng = np.random.default_rng(n[0])
    E = [rng.standard_normal(n).astype(np.float32) for _ in range(3)]
    pos = [rng.uniform(0, n[d], count).astype(np.float32) for d in range(3)]
    b = pi.Bunch(*[p * DX for p in pos], *np.zeros((3, count)), -pi.E_CHARGE, pi.M_E, 1.0)
    z = np.zeros(n)
    return native.Simulation(*n, DX, pi.courant_dt(DX), z, z, bc=(native.BC_PERIODIC,) * 3, init_E=E, bunch=b,
                             **kw), np.stack(E), np.stack(pos)


@pytest.mark.parametrize("n,count", [((3, 2, 2), 5), ((64, 32, 32), 1 << 16), ((65537, 1, 1), (1 << 16) + 1)])
@pytest.mark.parametrize("fields_first", [True, False])
def test_every_read_gives_the_state(n, count, fields_first):
    s, E, pos = _sim(n, count)
    for call in range(6):
        if fields_first or call:
            assert np.array_equal(s.fields(native.FIELD_E), E)
            assert not s.fields(native.FIELD_H).any()
        p = s.particles()
        assert np.abs(p[:3] / DX - pos).max() <= 2.0 ** -24 * 2 * max(n)


def test_fixed_point_current_reads_again():
    s, _, _ = _sim((65, 23, 22), 100, deposit_mode=2)  # 8-byte elements: 263 KB
    for _ in range(4):
        assert not s.fields(native.FIELD_JB).any()
