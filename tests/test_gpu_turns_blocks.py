"""XCDs taking turns at chunks of tiles against contiguous blocks, at sizes where the
reference shape (64 x 8 cells) has fewer than 1024 tiles and so runs in blocks, and the
others 1024 or more: the same arithmetic per cell, E, H and J_pol equal bit for bit."""
import numpy as np
import pytest

import pic_inputs as pi
from paper_1505_04007_amd import native

pytestmark = pytest.mark.gpu

P, C = native.BC_PERIODIC, native.BC_CPML


def _tiles(n, fx, fy):
    return -(-n[0] // fx) * -(-n[1] // fy) * n[2]


@pytest.mark.parametrize("n,bc", [
    ((128, 72, 56), (C, C, C)),    # 2016 runs: 15 rounds of 8 chunks and 96
    ((192, 40, 67), (P, P, C)),    # 2010, ragged chunks
    ((250, 137, 9), (P, C, P)),    # planes above 2^15 cells
])
def test_turns_equal_blocks(n, bc):
    rng = np.random.default_rng(sum(n))
    dx = 2e-9
    wp = np.where(rng.random(n) < 0.2, pi.AG_WP, 0.0)
    E = [rng.standard_normal(n) for _ in range(3)]
    assert _tiles(n, 64, 8) < 1024 <= min(_tiles(n, 64, 4), -(-n[0] * n[1] * n[2] // 256))
    got = {}
    for shape in (5, 3, 11, 0, 8):
        s = native.Simulation(*n, dx, pi.courant_dt(dx), wp, 0.01 * wp, bc=bc, npml=4, init_E=E)
        s.tune(force=shape)
        s.step(4)
        got[shape] = [s.fields(f) for f in (native.FIELD_E, native.FIELD_H, native.FIELD_JPOL)]
        s.close()
    for shape in (3, 11, 0, 8):
        for a, b in zip(got[5], got[shape]):
            assert np.array_equal(a, b), shape
