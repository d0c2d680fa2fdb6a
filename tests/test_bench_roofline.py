"""The bench line's roofline names the limit the kernel is nearer to, with the other
beside it."""
import pytest

import bench


@pytest.mark.parametrize("algo,valu,bound", [
    (1.5e9, 8.1e7, "hbm"),   # 0.69 of HBM, 0.48 of VALU issue
    (4.8e8, 1.25e8, "alu"),  # 0.22 and 0.74
    (1.5e9, None, "hbm"),    # no counters
])
def test_nearer_limit(algo, valu, bound):
    t = 2.75e-4
    r = bench.roofline("k", t, algo, {"valu_per_launch": valu, "bytes_per_launch": 5} if valu else {})
    frac = {"hbm": algo / t / 1e9 / bench.HBM_PEAK_GBS}
    if valu:
        frac["alu"] = valu / t / 1e9 / bench.VALU_PEAK_G
    assert r["bound"] == bound == max(frac, key=frac.get)
    assert abs(r["frac"] - frac[bound]) <= 1e-4
    assert r["unit"].startswith("GB/s" if bound == "hbm" else "G wave64")
    assert set(r) & {"hbm", "alu"} == set(frac) - {bound}
    for k in set(frac) - {bound}:
        assert abs(r[k]["frac"] - frac[k]) <= 1e-4
    assert r["kernel"] == "k" and r["traffic"] == (5 if valu else None)
