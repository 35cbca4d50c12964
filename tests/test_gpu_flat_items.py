"""bf16 tile maps whose items follow the planes' groups of 64 tile rows rather than the rows (widths of more than 32 tile columns that are no
multiple of 64): groups that are full, that end inside an item and that have fewer tiles than one item, rows that an item crosses once and
twice, widths that are and are not multiples of 8, in the plain encodes and decodes and in those with a basis gradient, of one matrix
and of two.

Bars: gpu_util.check (see test_gpu_any_width.py)."""
import numpy as np
import pytest

import stl_synth
from oracle import planes

pytestmark = pytest.mark.gpu

NAMES = ("dX", "dWhat", "dE_X", "dD")
# M, K, N tile counts, r
SHAPES = [(1, 33, 34, 5), (63, 36, 33, 3), (64, 63, 65, 8), (65, 100, 72, 33), (129, 127, 191, 49), (128, 40, 250, 16), (200, 200, 50, 32), (2, 130, 264, 64),
          (67, 1000, 48, 8), (1100, 37, 41, 32),
          # encodes and decodes without a basis gradient and pairs: from 2048 items of a row's 64 columns (4096 if the width is a multiple of 8) on
          (2100, 37, 41, 5), (4100, 40, 72, 3), (690, 164, 133, 49)]
PAIRS = [(28, 160, 148, 164, 8), (3, 2000, 1996, 140, 33)]


@pytest.fixture(scope="module")
def gu():
    import gpu_util
    return gpu_util


@pytest.mark.parametrize("M,K,N,r", SHAPES)
def test_step(gu, M, K, N, r):
    p = stl_synth.stl_problem(4 * M, 4 * K, 4 * N, r, seed=2300 + M + K + N + r, dtype="bf16", with_dC=True)
    got = gu.step(p, "bf16")
    C, Y = planes.forward(p["X"], p["What"], p["E_X"], p["D"], return_yhat=True)
    gu.check(got["C"], C, "bf16", "C")
    gu.check(got["Yhat"], Y, "bf16", "Yhat", slab=1)
    ref = dict(zip(NAMES, planes.backward(p["X"], p["What"], p["E_X"], p["D"], p["dC"])))
    for name in NAMES:
        gu.check(got[name], ref[name], "bf16", name)
    # planes are stored in whole groups of rows: what lies behind the last row, in those given and in the workspace's, is not a number
    # and reaches nothing
    grads = gu.backward(p, "bf16", yhat=got["Yhat"], xhat=got["Xhat"], poison=True)
    for name in NAMES:
        gu.check(grads[name], ref[name], "bf16", name)
    # the matrix gradient alone, and the basis gradients alone
    one = gu.backward(p, "bf16", skip=("dWhat", "dE_X", "dD"))
    two = gu.backward(p, "bf16", skip=("dX", "dWhat"))
    gu.check(one["dX"], ref["dX"], "bf16", "dX")
    for name in ("dE_X", "dD"):
        gu.check(two[name], ref[name], "bf16", name)


@pytest.mark.parametrize("transposed", [False, True])
@pytest.mark.parametrize("nb,m,k,n,r", PAIRS)
def test_pairs(gu, nb, m, k, n, r, transposed):
    p = stl_synth.aa_problem(nb, m, k, n, r, seed=2400 + m + r, dtype="bf16", with_dC=True)
    args = (p["A"], p["B"], p["E_A"], p["E_B"], p["D"])
    if transposed:
        args = (p["A"], np.concatenate([b.T for b in np.split(p["B"], nb)]), p["E_A"], p["E_B"], p["D"])
    ref = planes.aa_backward(*args, p["dC"], nbatch=nb, b_transposed=transposed)
    C = planes.aa_forward(*args, nbatch=nb, b_transposed=transposed)
    kw = {"flags": gu.stl.STL_FLAG_B_TRANSPOSED if transposed else 0}
    gu.check(gu.aa_forward(*args, nb, "bf16", **kw), C, "bf16", "C")
    got = gu.aa_backward(*args, p["dC"], nb, "bf16", **kw)
    for name, want in zip(("dA", "dB", "dE_A", "dE_B", "dD"), ref):
        gu.check(got[name], want, "bf16", name)
