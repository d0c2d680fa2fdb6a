"""Probe spectra, sampled by the next step's H update or at a call's end: every
step counted once whatever the calls' lengths, and the phases' sine and cosine.

The recorded series holds the Ez each sample used, so the DFT is recomputed
from it in FP64.  A phase w t is rounded once on either side alike; sine and
cosine, a product and an addition per term are within 4 units of 2^-53 each, so
a sum differs by at most 1e-15 of the sum of |dt Ez| per term."""
import numpy as np
import pytest

import pic_inputs as pi
from paper_1505_04007_amd import native

pytestmark = pytest.mark.gpu


def _sim(omega, nprobe, **kw):
    n, dx = (20, 14, 12), 4e-9
    rng = np.random.default_rng(5)
    wp, g = pi.film_maps(*n, 3, 6)
    E = [rng.standard_normal(n) for _ in range(3)]
    pr = np.array([[(2 + p % 16) * dx, (1 + p % 11) * dx, (1.5 + p % 9) * dx] for p in range(nprobe)])
    return native.Simulation(*n, dx, pi.courant_dt(dx), wp, g, bc=(1, 0, 2), npml=3, init_E=E, probes=pr, omega=omega,
                             series_len=100, **kw)


@pytest.mark.parametrize("nprobe,omega", [
    (1, [0.0]),
    (3, np.linspace(0.3, 1.0, 64) * pi.AG_WP),
    (256, [1e15, -3e16, 7e18]),            # more probes than a tile of 128 threads
    (2, [1e20, 1e22, 2.5e23, -1e23]),      # phases up to 6e7
])
@pytest.mark.parametrize("calls", [[60], [1] * 60, [1, 2, 57], [0, 59, 0, 1]])
def test_spectra_from_the_series(nprobe, omega, calls):
    s = _sim(omega, nprobe)
    if len(calls) == 3:
        s.tune(force=1)
    for c in calls:
        s.step(c)
    F, ser = s.probe(series=True)
    ez = ser[:60 * nprobe].reshape(60, nprobe)
    t = np.arange(1, 61) * s.dt
    ph = np.multiply.outer(np.asarray(omega, dtype=float), t)
    want = s.dt * (np.cos(ph) @ ez - 1j * (np.sin(ph) @ ez)).T
    bound = 60e-15 * s.dt * np.abs(ez).sum(axis=0)
    assert np.all(np.abs(F - want) <= bound[:, None])


@pytest.mark.parametrize("use_graph", [False, True])
def test_batch_counts_every_step_once(use_graph):
    om = np.linspace(0.3, 1.0, 8) * pi.AG_WP
    a, b = _sim(om, 3), _sim(om, 3)
    batch = native.Batch([a], use_graph=use_graph)
    for c in (1, 10, 23, 26):
        batch.step(c)
    b.step(60)
    assert np.array_equal(a.probe(), b.probe())
    a.step(3)
    b.step(3)
    assert np.array_equal(a.probe(), b.probe())
