"""Ragged backward with everything saved and asked for (the last tile rows in one pass over dC, the three sums in one launch) against the
oracle and, bit for bit, against the call that recomputes its planes; widths of fewer than 8 tiles, which take the general path,
two tile rows per image, and more partial sums than one workgroup of the last pass reads at once.

Bars: gpu_util.TOL, relative Frobenius error (see test_gpu_ragged.py)."""
import numpy as np
import pytest

import stl_synth
from oracle import planes

pytestmark = pytest.mark.gpu

NAMES = ("dX", "dWhat", "dE_X", "dD", "dfold")


@pytest.fixture(scope="module")
def gu():
    import gpu_util
    return gpu_util


@pytest.mark.parametrize("nimg,rows,k,n,r", [(3, 9, 32, 32, 64), (2, 7, 32, 36, 1), (5, 6, 20, 28, 33), (16, 50, 192, 1088, 49), (33, 21, 520, 260, 17)])
def test_saved(gu, nimg, rows, k, n, r):
    p = stl_synth.ragged_problem(nimg, rows, k, n, r, seed=9300 + rows + k + n + r, dtype="bf16", with_dC=True)
    ref = dict(zip(NAMES, planes.ragged_backward(p["X"], p["What"], p["E_X"], p["D"], p["fold"], p["dC"], rows)))
    _, Xh, Yh = gu.ragged_forward(p, rows, "bf16", save=True)
    base = gu.ragged_backward(p, rows, "bf16")
    saved = gu.ragged_backward(p, rows, "bf16", saved=(Xh, Yh))
    for name in NAMES:
        assert gu.rel(saved[name], ref[name]) <= gu.TOL["bf16"], name
        assert np.array_equal(saved[name], base[name]), name
