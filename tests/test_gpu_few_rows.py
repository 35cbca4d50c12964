"""Plane products of few rows (stl_gemm_rows.hip): 1, 7, 8, 16, 17, 32 and 33 tile rows; contractions of fewer chunks (32) than wavefronts, of a whole
number of rounds and of one chunk more, ending inside a chunk; widths of one, of whole and of incomplete blocks; both block
widths (at most 256 blocks of 64 columns, and more) and both sides of the rule for more than 16 rows.  test_cpu_routes.py asserts that these
shapes reach every form of the kernel.

Bars: gpu_util.check (see test_gpu_any_width.py); one entry's bar needs r K of 72 and more (see test_gpu_staged.py)."""
import numpy as np
import pytest

import stl_synth
from oracle import planes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gu():
    import gpu_util
    return gpu_util


SHAPES = [(8, 8, 16, 9), (16, 264, 136, 49), (9, 1000, 248, 8), (15, 296, 1016, 64), (1, 776, 56, 40), (7, 1000, 248, 8), (16, 512, 64, 3),
          (13, 256, 1032, 32), (32, 128, 128, 5), (17, 136, 1032, 9), (31, 520, 1024, 32), (17, 2048, 56, 4), (32, 128, 1024, 32), (17, 160, 1032, 17)]
OTHERS = [(32, 120, 128, 5), (33, 128, 128, 5)]                       # on the far side of the rule


@pytest.mark.parametrize("M,K,N,r", SHAPES + OTHERS)
def test_few_rows(gu, M, K, N, r):
    p = stl_synth.stl_problem(4 * M, 4 * K, 4 * N, r, seed=1700 + M + K + N + r, dtype="bf16", with_dC=True)
    got = gu.step(p, "bf16")
    C, Y = planes.forward(p["X"], p["What"], p["E_X"], p["D"], return_yhat=True)
    gu.check(got["Yhat"], Y, "bf16", "Yhat", slab=1)
    gu.check(got["C"], C, "bf16", "C")


@pytest.mark.parametrize("M,K,N,r", [(16, 64, 72, 9), (5, 40, 264, 33), (16, 72, 64, 9)])
def test_single_pair_of_activations(gu, M, K, N, r):
    """A second operand in the grouped layout: one group of up to 64 tile rows is taken here, more are not."""
    p = stl_synth.aa_problem(1, 4 * M, 4 * K, 4 * N, r, seed=1800 + M + K + N + r, dtype="bf16")
    args = (p["A"], p["B"], p["E_A"], p["E_B"], p["D"])
    gu.check(gu.aa_forward(*args, 1, "bf16"), planes.aa_forward(*args, nbatch=1), "bf16", "C")


@pytest.mark.parametrize("M,K,N,r", [(16, 40, 72, 3), (9, 1000, 248, 8), (20, 136, 264, 5), (18, 160, 1032, 17), (15, 264, 1032, 32), (31, 168, 1032, 17)])
def test_infinities_at_the_end_of_the_contraction(gu, M, K, N, r):
    """One infinity in the last contraction element of each operand makes one row and one column of its plane infinite, never NaN, and
    leaves every other entry as it was: the elements that are read again to fill the last chunk take no part."""
    import torch

    import paper_2503_12211_amd as stl
    rng = np.random.default_rng(M + K + N)
    X = stl_synth.round_to(rng.standard_normal((r, M, K)), "bf16")
    W = stl_synth.round_to(rng.standard_normal((r, K, N)), "bf16")
    prob = stl.Problem(4 * M, 4 * K, 4 * N, r)

    def multiply(X, W):
        gd = gu.Guard()
        Y = gd.alloc((stl.stl_plane_elems(M, N, r),), torch.bfloat16)
        stl.stl_plane_matmul(prob, gu.planes_to_dev(X, "bf16"), gu.dev(W, "bf16"), Y)
        gd.check()
        return gu.planes_to_host(Y, r, M, N)
    clean = multiply(X, W)
    Xi, Wi = X.copy(), W.copy()
    Xi[0, M // 2, K - 1] = np.inf
    Wi[1, K - 1, N // 3] = -np.inf
    want = clean.copy()
    want[0, M // 2] = np.where(W[0, K - 1] > 0, np.inf, -np.inf)
    want[1, :, N // 3] = np.where(X[1, :, K - 1] > 0, -np.inf, np.inf)
    assert np.array_equal(multiply(Xi, Wi), want)
