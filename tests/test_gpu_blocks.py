"""bf16 plane products over all their block sizes (256 x 256, 128 x 256, 128 x 128, 64 x 64), with blocks that hang over the edge
and contractions that end inside a stage of 32 (and, in the weight gradient, at any tile row).

Bars: gpu_util.check (see test_gpu_any_width.py)."""
import numpy as np
import pytest

import stl_synth
from oracle import planes

pytestmark = pytest.mark.gpu

NAMES = ("dX", "dWhat", "dE_X", "dD")


@pytest.fixture(scope="module")
def gu():
    import gpu_util
    return gpu_util


# M, K, N tile counts, r -- blocks of the three products Yhat, dXhat, dWhat
SHAPES = [(16, 40, 64, 8),          # 64 or 128, 128, 128; fewer rows than a block
          (300, 200, 264, 3),       # 64, 64, 64
          (130, 72, 136, 49),       # 128, 64, 128
          (257, 488, 520, 40),      # 128, 128 x 256, 128; the weight gradient contracts over an odd number of rows
          (640, 320, 512, 24),      # 128 x 256, 128, 128
          (520, 264, 776, 32),      # 128, 128, 256
          (1030, 72, 520, 64),      # 128, 128, 128 x 256
          (2040, 232, 2040, 4)]     # 256 with a contraction of 232; 128 for the others


@pytest.mark.parametrize("M,K,N,r", SHAPES)
def test_step_blocks(gu, M, K, N, r):
    p = stl_synth.stl_problem(4 * M, 4 * K, 4 * N, r, seed=700 + M + K + N + r, dtype="bf16", with_dC=True)
    got = gu.step(p, "bf16")
    C, Y = planes.forward(p["X"], p["What"], p["E_X"], p["D"], return_yhat=True)
    gu.check(got["C"], C, "bf16", "C")
    gu.check(got["Yhat"], Y, "bf16", "Yhat", slab=1)
    ref = dict(zip(NAMES, planes.backward(p["X"], p["What"], p["E_X"], p["D"], p["dC"])))
    for name in NAMES:
        gu.check(got[name], ref[name], "bf16", name)
    init = [np.ones_like(ref[nm], dtype=np.float32) for nm in NAMES[1:]]
    acc = gu.backward(p, "bf16", accumulate=1, init=init)
    # one rounding of (1 + gradient) on top of the same sums
    assert np.abs(acc["dWhat"] - 1.0 - got["dWhat"]).max() <= 2.0 ** -22 * max(1.0, np.abs(got["dWhat"]).max())


@pytest.mark.parametrize("M,K,N,r", [(130, 72, 136, 9), (300, 40, 264, 5), (70, 250, 262, 4)])
def test_non_finite_rows_stay_where_they_are(gu, M, K, N, r):
    """Infinities and NaN in one tile row of X reach that tile row of C and no other: nothing of a neighbouring row, or of
    what lies beyond the contraction's end, enters a product."""
    p = stl_synth.stl_problem(4 * M, 4 * K, 4 * N, r, seed=800 + M, dtype="bf16")
    clean = gu.forward(p, "bf16")
    q = dict(p, X=p["X"].copy())
    row = M // 2
    q["X"][4 * row] = np.inf
    q["X"][4 * row + 1] = np.nan
    got = gu.forward(q, "bf16")
    others = np.r_[0:4 * row, 4 * row + 4:4 * M]
    assert np.array_equal(got[others], clean[others])
    assert not np.isfinite(got[4 * row:4 * row + 4]).all()
