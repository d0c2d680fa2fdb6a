"""native.DEFAULT_TILE is the shape pic_init gives a grid, and what the bench keeps when
it does not tune."""
import os
import re

from paper_1505_04007_amd import native

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _read(*path):
    return open(os.path.join(ROOT, *path)).read()


def test_default_tile_is_the_librarys():
    src = _read("paper_1505_04007_amd", "csrc", "pic_internal.hpp")
    name = re.search(r"constexpr int DEFAULT_TILE = (\w+);", src).group(1)
    assert int(re.search(rf"constexpr int {name} = (\d+)", src).group(1)) == native.DEFAULT_TILE


def test_bench_without_tuning_keeps_it():
    assert set(re.findall(r"tune\(force=([\w.]+)\)", _read("bench.py"))) == {"native.DEFAULT_TILE"}
