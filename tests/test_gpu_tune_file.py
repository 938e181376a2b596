"""GPU: the tile-choice file (TNC_AUTOTUNE_CACHE).

A line counts only if it was measured on the kernels that the library has now;
a line of other kernels, or one that cannot be read, is passed over, and the
lines after it still count.
"""
import os
import re

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2606_01852_amd import tnc  # noqa: E402

SHAPE = (4, 1024, 512, 64)   # h, m, n, k (too short for split K)


def chosen(monkeypatch, path):
    monkeypatch.setenv("TNC_AUTOTUNE_CACHE", str(path))
    ctx = tnc.Context(0, arena_bytes=1 << 30)
    h, m, n, k = SHAPE
    leaves = [np.zeros(s, np.complex64) for s in ((h, m, k), (h, n, k))]
    net = tnc.Network(ctx, [(0, 1, 3), (0, 2, 3)], np.array([h, m, n, k], dtype=np.int64), (0, 1, 2), leaves)
    plan = tnc.Plan(net, [(0, 1)])
    v = tnc.tnc_plan_get_step(plan.handle, 0).variant
    plan.close()
    net.close()
    ctx.close()
    return v


def generation():
    """The number that the library writes before the precision of a line."""
    src = os.path.join(os.path.dirname(tnc.__file__), "csrc", "autotune.cpp")
    return int(re.search(r"kTuneGeneration = (\d+)", open(src).read()).group(1))


@pytest.mark.parametrize("first", ["0", "{old}:0", "{new}:", "x", ""])
def test_other_kernels_lines_do_not_count(monkeypatch, tmp_path, first):
    path, g = tmp_path / "tune.txt", generation()
    h, m, n, k = SHAPE
    default = chosen(monkeypatch, tmp_path / "none.txt")
    other = 5 if default != 5 else 4
    first = first.format(old=g - 1, new=g)
    path.write_text(f"{first} 0 0 {h} {m} {n} {k} {other}\n")
    assert chosen(monkeypatch, path) == default
    path.write_text(f"{first} 0 0 {h} {m} {n} {k} {other}\n{g}:0 0 0 {h} {m} {n} {k} {other}\n")
    assert chosen(monkeypatch, path) == other
