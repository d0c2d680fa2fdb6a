"""Maps and fields in and out: arrays of any order and type, sizes around the
pieces they are moved in, and the particles' load order.  Values are moved, not
computed: no tolerance beyond the FP32 state's rounding of the input."""
import numpy as np
import pytest

import pic_inputs as pi
from paper_1505_04007_amd import native


@pytest.mark.parametrize("n", [(1, 1, 1), (15, 2, 3), (16, 1, 4), (17, 5, 2), (64, 3, 3), (0, 2, 2)])
@pytest.mark.parametrize("make", [
    lambda a: a, np.asfortranarray, lambda a: a.astype(np.float32), lambda a: (8 * a).astype(int),
    lambda a: np.repeat(a, 2, axis=1)[:, ::2], lambda a: a[::-1], lambda a: a.tolist() if a.size else a])
def test_to_compact(n, make):
    a = make(np.random.default_rng(3).random(n))
    want = np.ascontiguousarray(np.asarray(a).transpose(2, 1, 0), dtype=np.float64)
    got = native.to_compact(a)
    assert got.dtype == np.float64 and got.flags.c_contiguous and np.array_equal(got, want)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [(1, 1, 1), (20, 7, 9), (128, 128, 64), (128, 129, 64), (257, 130, 63)])
def test_fields_come_back(n):  # the piece is 2^20 values: below, at and above it, and two pieces and some
    rng = np.random.default_rng(1)
    E = [rng.standard_normal(n).astype(np.float32) for _ in range(3)]
    z = np.zeros(n)
    s = native.Simulation(*n, 2e-9, pi.courant_dt(2e-9), z, z, bc=(native.BC_PERIODIC,) * 3, init_E=E)
    assert np.array_equal(s.fields(native.FIELD_E), np.stack(E).astype(np.float64))
    assert not s.fields(native.FIELD_H).any()


@pytest.mark.gpu
@pytest.mark.parametrize("count", [1, 2, 3000, 1 << 20, (1 << 20) + 5])
def test_particles_come_back_in_their_order(count):
    n, dx = (40, 6, 5), 2e-9
    rng = np.random.default_rng(count)
    pos = [rng.uniform(0, n[d], count).astype(np.float32) for d in range(3)]
    pos[0][::7] = pos[0][0]  # equal keys
    u = rng.standard_normal((3, count)) * 1e7
    b = pi.Bunch(*[p * dx for p in pos], *u, -pi.E_CHARGE, pi.M_E, 1.0)
    z = np.zeros(n)
    s = native.Simulation(*n, dx, pi.courant_dt(dx), z, z, bc=(native.BC_PERIODIC,) * 3, bunch=b)
    p = s.particles()
    for d in range(3):
        assert np.abs(p[d] / dx - pos[d]).max() <= 2.0 ** -24 * 2 * n[d]
        assert np.abs(p[3 + d] - u[d]).max() <= 2.0 ** -23 * np.abs(u[d]).max()
