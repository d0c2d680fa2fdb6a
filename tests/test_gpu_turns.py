"""Field and adjoint kernels with the XCDs taking turns at chunks of tiles: from
1024 tiles on where the last axis of the order has absorbing slabs or a plane is
large.  The map from
workgroups to tiles is a permutation that must reach every cell once, at whole
rounds of 8 chunks and with any remainder; the same cells in tiles of 512 (fewer
than 1024 of them) are updated in contiguous blocks, with the same arithmetic, so E, H
and J_pol are equal bit for bit.  The adjoint has one shape and is compared with the
oracle, at the bars of fields-only gradients (1e-5)."""
import numpy as np
import pytest

import pic_inputs as pi
import test_gpu_grad as tg
from paper_1505_04007_amd import native

pytestmark = pytest.mark.gpu

P, C = native.BC_PERIODIC, native.BC_CPML


@pytest.mark.parametrize("n,bc", [
    ((64, 64, 64), (P, C, C)),     # 1024 tiles: whole rounds
    ((64, 64, 65), (P, P, C)),     # 1040
    ((61, 67, 65), (C, C, C)),     # 1038 and a ragged last run
    ((64, 80, 71), (P, C, P)),     # the slabs along y: turns for bands only
    ((128, 72, 64), (C, C, C)),    # 2304 = 2 rounds and 256
    ((256, 132, 10), (P, P, P)),   # planes above 2^15 cells, no slabs
])
def test_turns_equal_blocks(n, bc):
    rng = np.random.default_rng(sum(n))
    dx = 2e-9
    wp = np.where(rng.random(n) < 0.2, pi.AG_WP, 0.0)
    E = [rng.standard_normal(n) for _ in range(3)]
    got = {}
    for shape in (5, 3, 11, 0, 8):
        s = native.Simulation(*n, dx, pi.courant_dt(dx), wp, 0.01 * wp, bc=bc, npml=4, init_E=E)
        s.tune(force=shape)
        s.step(4)
        got[shape] = [s.fields(f) for f in (native.FIELD_E, native.FIELD_H, native.FIELD_JPOL)]
    for shape in (3, 11, 0, 8):
        for a, b in zip(got[5], got[shape]):
            assert np.array_equal(a, b), shape


@pytest.mark.parametrize("n", [(64, 64, 64), (66, 64, 65)])
def test_gradient_over_the_whole_grid(n):
    dx, N = 2e-9, 10
    rng = np.random.default_rng(n[0])
    wp, g = pi.film_maps(*n, 5, n[2] - 6)
    probes = np.array([[rng.uniform(1, n[d] - 1) * dx for d in range(3)] for _ in range(200)])
    w = pi.Workload("grad_turns", *n, dx, pi.courant_dt(dx), (P, P, C), 4, wp, g, None, probes,
                    np.array([0.68 * pi.AG_WP]), N)
    E = []
    for c in range(3):
        e = 1e6 * rng.standard_normal([n[a] + (a != c) for a in range(3)])
        for a in range(3):
            lo, hi = [slice(None)] * 3, [slice(None)] * 3
            lo[a], hi[a] = 0, n[a]
            if a != c and w.bc[a] == P:
                e[tuple(hi)] = e[tuple(lo)]
            elif a != c:
                e[tuple(lo)] = e[tuple(hi)] = 0.0
        E.append(e)
    o = tg._oracle(w, E)
    Lo, gwo, ggo = o.grad(N, w.omega[0])
    L, gw, gg = tg._gpu(w, E).grad(w.omega[0], N)
    assert abs(L - Lo) <= 1e-5 * Lo
    assert tg._rel(gw, gwo) <= 1e-5 and tg._rel(gg, ggo) <= 1e-5
