"""Plane products of few rows (stl_gemm_rows.hip): 1, 7, 8, 16, 17, 32 and 33 tile rows; contractions of fewer chunks (32) than wavefronts, of a whole
number of rounds and of one chunk more, ending inside a chunk; widths of one, of whole and of incomplete blocks; both block
widths (at most 256 blocks of 64 columns, and more) and both sides of the rule for more than 16 rows.

Bars: gpu_util.check (see test_gpu_any_width.py); one entry's bar needs r K of 72 and more (see test_gpu_staged.py)."""
import pytest

import stl_synth
from oracle import planes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gu():
    import gpu_util
    return gpu_util


@pytest.mark.parametrize("M,K,N,r", [(8, 8, 16, 9), (16, 264, 136, 49), (9, 1000, 248, 8), (15, 296, 1016, 64), (1, 776, 56, 40), (7, 1000, 248, 8), (16, 512, 64, 3),
                                     (13, 256, 1032, 32), (32, 128, 128, 5), (17, 136, 1032, 9), (31, 520, 1024, 32), (17, 2048, 56, 4), (32, 120, 128, 5),
                                     (33, 128, 128, 5)])
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
