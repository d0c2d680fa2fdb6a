"""Probe spectra at phases of any size: the DFT's sine and cosine are right to
rounding from omega t below 1 to 1e280, where the reduction by pi/2 takes its other
way (from 2^45 on).  Against the sums of the recorded samples with the C library's
sine and cosine of the same FP64 phases: a term's two factors and their product are
off by at most 4 roundings of 1.1e-16, and 6 terms' sum by 5, so 1e-15 of the sum of
dt |Ez|."""
import math

import numpy as np
import pytest

import pic_inputs as pi
from paper_1505_04007_amd import native

pytestmark = pytest.mark.gpu

N, DX, STEPS = (12, 10, 9), 2e-9, 6
DT = pi.courant_dt(DX)
EDGE = 2.0 ** 45 / (3 * DT)  # the phase of step 3 lies on the border
OMEGA = np.concatenate([np.array([0.0, 0.3, -1.7, 1e3, 1e9, 2.0 ** 30, 1e15, -1e17, 1e22, 1e60, -3e140, 1e280]) / DT,
                        [EDGE, np.nextafter(EDGE, 0), np.nextafter(EDGE, np.inf), -EDGE]])


BELOW = np.array([0.0, 1e-3, -2.5, np.nextafter(4.0, 0)]) / DT  # all of a step's phase below 4: no large ones


@pytest.mark.parametrize("omega", [OMEGA, BELOW, np.append(BELOW, 4.0 / DT)])
@pytest.mark.parametrize("how", ["one call", "step by step", "batch", "one sweep"])
def test_spectra_at_any_phase(how, omega):
    rng = np.random.default_rng(3)
    E = [rng.standard_normal(N) for _ in range(3)]
    z = np.zeros(N)
    probes = np.array([[4.5, 4.5, 4.5], [7.0, 2.0, 3.0], [2.0, 6.0, 5.0]]) * DX
    s = native.Simulation(*N, DX, DT, z, z, probes=probes, omega=omega, series_len=STEPS, init_E=E,
                          field_sweep=int(how == "one sweep"))
    if how == "batch":
        native.Batch([s]).step(STEPS)
    elif how == "step by step":
        for _ in range(STEPS):
            s.step(1)
    else:
        s.step(STEPS)
    F, ser = s.probe(series=True)
    ser = ser.reshape(STEPS, len(probes))
    assert np.abs(ser).max() > 0
    for p in range(len(probes)):
        bound = 1e-15 * np.sum(np.abs(ser[:, p])) * DT
        for m, w in enumerate(omega):
            ph = [float(w) * (n * DT) for n in range(1, STEPS + 1)]
            re = math.fsum(DT * ser[n, p] * math.cos(ph[n]) for n in range(STEPS))
            im = math.fsum(-DT * ser[n, p] * math.sin(ph[n]) for n in range(STEPS))
            assert abs(F[p, m].real - re) <= bound and abs(F[p, m].imag - im) <= bound, (w, F[p, m], re, im)
