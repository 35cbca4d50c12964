"""Register-staged plane products where their stages, groups and chunks end: contractions of one stage (64) and of one piece (32), of
4, 5, 12 and 13 stages over two and four groups of wavefronts, rows whose last chunk has one element, stacked problems whose
rows straddle the planes' groups of 64, thin outputs of widths that are multiples of 8.  test_cpu_routes.py asserts which groups they reach.

Bars: gpu_util.check (see test_gpu_any_width.py).  Its bar for one entry takes an entry as the sum of many terms: with r planes and
a contraction of K the entry's own scale has a relative spread of about sqrt(2 / (r K)), so that over 1e6 entries (4.9 sigma) the largest
error is 2.9e-3 * 4.9 * (1 + 4.9 * sqrt(2 / (r K))): 0.026 at r K = 72, but 0.038 at r K = 18 with tails that are no longer normal (0.0501
was seen at 2 x (257 x 9 x 321), r = 2).  Stacked shapes, all checked entry by entry over 1e5 and more entries, have r K >= 72."""
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


# M, K, N, r: every dimension is the contraction of one of the three products
SHAPES = [(31, 32, 33, 3), (63, 64, 65, 2), (193, 257, 9, 5), (17, 705, 769, 4), (705, 9, 67, 3), (833, 65, 17, 8), (70, 193, 129, 49)]
STACKED = [(9, 50, 16, 50, 8, True), (5, 33, 9, 31, 49, False), (3, 64, 16, 64, 32, True), (3, 48, 64, 24, 5, False), (2, 257, 9, 321, 8, True),
           (1, 705, 66, 67, 3, False), (1, 833, 67, 65, 3, True)]        # the last two: four groups store the gradient of the second operand


@pytest.mark.parametrize("M,K,N,r", SHAPES)
def test_step_staged(gu, M, K, N, r):
    p = stl_synth.stl_problem(4 * M, 4 * K, 4 * N, r, seed=400 + M + K + N + r, dtype="bf16", with_dC=True)
    got = gu.step(p, "bf16")
    _, Y = planes.forward(p["X"], p["What"], p["E_X"], p["D"], return_yhat=True)
    gu.check(got["Yhat"], Y, "bf16", "Yhat", slab=1)
    ref = dict(zip(NAMES, planes.backward(p["X"], p["What"], p["E_X"], p["D"], p["dC"])))
    for name in NAMES:
        gu.check(got[name], ref[name], "bf16", name)
    init = [np.ones_like(ref[nm], dtype=np.float32) for nm in NAMES[1:]]
    acc = gu.backward(p, "bf16", accumulate=1, init=init)
    assert np.abs(acc["dWhat"] - 1.0 - got["dWhat"]).max() <= 2.0 ** -22 * max(1.0, np.abs(got["dWhat"]).max())


@pytest.mark.parametrize("nb,M,K,N,r,bt", STACKED)
def test_stacked_staged(gu, nb, M, K, N, r, bt):
    import paper_2503_12211_amd as stl
    fl = stl.STL_FLAG_B_TRANSPOSED if bt else 0
    p = stl_synth.aa_problem(nb, 4 * M, 4 * K, 4 * N, r, seed=500 + M + K + N + r, dtype="bf16", with_dC=True)
    B = p["B"]
    if bt:
        B = np.ascontiguousarray(np.concatenate([B[b * 4 * K:(b + 1) * 4 * K].T for b in range(nb)], axis=0))
    args = (p["A"], B, p["E_A"], p["E_B"], p["D"])
    gu.check(gu.aa_forward(*args, nb, "bf16", flags=fl), planes.aa_forward(*args, nbatch=nb, b_transposed=bt), "bf16", "C")
    got = gu.aa_backward(*args, p["dC"], nb, "bf16", flags=fl)
    ref = dict(zip(("dA", "dB", "dE_A", "dE_B", "dD"), planes.aa_backward(*args, p["dC"], nbatch=nb, b_transposed=bt)))
    for name in ref:
        gu.check(got[name], ref[name], "bf16", name)
