"""A batch whose tuning ends in an error steps on as before.

A member of 1x3x2^23 cells has 98304 runs of 256 cells and 2^23 tiles of 64x4
cells, but 2^24 of 64x2, one more than a batch can number: the tuner gives up at
the second shape it times.  The batch must then be back on the shape it was
created with, for direct launches and for the graph captured before, with the
step clock running: E equals the member's stepped alone, bit for bit."""
import numpy as np
import pytest

import pic_inputs as pi
from paper_1505_04007_amd import native

pytestmark = pytest.mark.gpu

N = (1, 3, 1 << 23)
STEPS = 12  # one replay of the graph's 10 steps and two direct ones


def _sim():
    rng = np.random.default_rng(5)
    # one random stretch repeated: not the same between any two neighbours
    E = [np.tile(rng.standard_normal((1, 3, 1 << 13)), (1, 1, 1 << 10)) for _ in range(3)]
    z = np.zeros(N)
    return native.Simulation(*N, 2e-9, pi.courant_dt(2e-9), z, z, bc=(native.BC_PERIODIC,) * 3, init_E=E)


def test_a_failed_tuning_changes_nothing():
    s = _sim()
    s.step(STEPS)
    want = s.fields(native.FIELD_E)
    s.close()
    for graph in (False, True):
        s = _sim()
        b = native.Batch([s], use_graph=graph)
        with pytest.raises(native.PicError) as e:
            b.tune(reps=1)
        assert e.value.status == native.PIC_EINVAL and "too many field tiles" in str(e.value)
        b.step(STEPS)
        assert s.stats()["steps"] == STEPS
        assert np.array_equal(s.fields(native.FIELD_E), want), graph
        b.close()
        s.close()
