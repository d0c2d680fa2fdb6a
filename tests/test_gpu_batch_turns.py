"""Batched field launches with the XCDs in blocks (no member has thick slabs or large
planes) and in turns (one has), at 1024 units and more and any remainder, for each tile
order: every member's fields equal its plain run's bit for bit."""
import numpy as np
import pytest

import pic_inputs as pi
from paper_1505_04007_amd import native

pytestmark = pytest.mark.gpu

P, C = native.BC_PERIODIC, native.BC_CPML


def _sim(n, bc, seed):
    rng = np.random.default_rng(seed)
    wp = np.where(rng.random(n) < 0.2, pi.AG_WP, 0.0)
    return native.Simulation(*n, 2e-9, pi.courant_dt(2e-9), wp, 0.01 * wp, bc=bc, npml=4,
                             init_E=[rng.standard_normal(n) for _ in range(3)])


@pytest.mark.parametrize("members", [
    [((64, 64, 65), (P, P, P)), ((61, 50, 33), (P, P, P)), ((40, 30, 37), (C, C, P))],  # blocks
    [((64, 64, 65), (P, P, P)), ((61, 50, 33), (P, P, P)), ((40, 30, 37), (P, P, C))],  # turns: the last one's slabs
    [((250, 140, 9), (P, P, P)), ((33, 20, 21), (P, P, P))],                            # turns: the first one's planes
])
@pytest.mark.parametrize("graph", [True, False])
@pytest.mark.parametrize("shape", [None, 0, 11])
def test_members_equal_plain_runs(members, graph, shape):
    got = []
    for batch in (False, True):
        S = [_sim(n, bc, q) for q, (n, bc) in enumerate(members)]
        if batch:
            b = native.Batch(S, use_graph=graph)
            if shape is not None:
                b.tune(force=shape)
            b.step(11)
        else:
            for s in S:
                s.step(11)
        got.append([s.fields(f) for s in S for f in (native.FIELD_E, native.FIELD_H, native.FIELD_JPOL)])
    for a, c in zip(*got):
        assert np.array_equal(a, c)
