"""The layout change of host arrays: the same values as numpy's copy on either way it
can take (whole rows, steps of x planes), and no slower than that copy where small
planes make many steps of 16 planes each a Python iteration (a factor of 5 when they
were; 2 is asked for, best of 5)."""
import time

import numpy as np
import pytest

from paper_1505_04007_amd import native


@pytest.mark.parametrize("n", [(1, 1, 1), (3, 0, 2), (91, 45, 53), (40, 16, 16), (33, 16, 32), (1023, 3, 5), (1024, 3, 5),
                               (1025, 1, 1), (2500, 2, 7), (1300, 40, 9)])
@pytest.mark.parametrize("kind", ["f8", "f4", "i4", "strided", "fortran"])
def test_values(n, kind):
    rng = np.random.default_rng(sum(n))
    a = rng.integers(-1000, 1000, n)
    a = a.astype({"f4": np.float32, "i4": np.int32}.get(kind, np.float64))
    if kind == "strided":
        a = np.repeat(a, 2, axis=1)[:, ::2][::-1]
    elif kind == "fortran":
        a = np.asfortranarray(a)
    got = native.to_compact(a)
    assert got.dtype == np.float64 and got.flags.c_contiguous and got.shape == n[::-1]
    assert np.array_equal(got, a.transpose(2, 1, 0))


def _best(f):
    t = []
    for _ in range(5):
        t0 = time.perf_counter()
        f()
        t.append(time.perf_counter() - t0)
    return min(t)


def test_long_thin_grids_take_no_longer_than_a_copy():
    a = np.random.default_rng(1).random((1 << 19, 2, 2))
    plain = _best(lambda: np.ascontiguousarray(a.transpose(2, 1, 0)))
    assert _best(lambda: native.to_compact(a)) <= 2 * plain
