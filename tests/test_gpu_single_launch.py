"""The single-launch forward and the decode-in-epilogue variant at the edges of their ring of stages: contractions of fewer stages than the
ring holds, of exactly as many and of more, ranks on either side of 8, 16 and 32 planes, incomplete blocks in both directions; and
the automatic choice on either side of its rule.

Bars: gpu_util.check (see test_gpu_any_width.py)."""
import numpy as np
import pytest

import stl_synth
from oracle import planes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gu():
    import gpu_util
    return gpu_util


@pytest.mark.parametrize("M,K,N,r", [(1, 16, 8, 1), (5, 32, 40, 8), (33, 48, 64, 7), (31, 64, 32, 9), (64, 80, 72, 16), (40, 96, 24, 15), (32, 112, 96, 17),
                                     (70, 16, 136, 32), (96, 128, 32, 32), (3, 320, 8, 24)])
def test_block_variants(gu, M, K, N, r):
    import paper_2503_12211_amd as stl
    p = stl_synth.stl_problem(4 * M, 4 * K, 4 * N, r, seed=1100 + M + K + N + r, dtype="bf16")
    C = planes.forward(p["X"], p["What"], p["E_X"], p["D"])
    rms = np.sqrt(np.mean(C ** 2))
    for flag in (stl.STL_FLAG_FUSED, stl.STL_FLAG_EPILOGUE, stl.STL_FLAG_AUTO):
        got = gu.forward(p, "bf16", flags=flag)
        assert gu.rel(got, C) <= gu.TOL["bf16"], flag
        assert np.abs(got - C).max() <= gu.ENTRY_C["bf16"] * max(rms, 1e-30) or r * K < 64, flag


@pytest.mark.parametrize("M,K,N,r,single", [(512, 112, 512, 16, True), (513, 112, 512, 16, False), (64, 128, 2048, 12, False), (512, 48, 512, 32, True),
                                            (64, 64, 512, 32, False), (64, 48, 512, 33, False)])
def test_automatic_choice(gu, M, K, N, r, single):
    """The automatic choice returns, bit for bit, what the variant that its rule names returns."""
    import paper_2503_12211_amd as stl
    p = stl_synth.stl_problem(4 * M, 4 * K, 4 * N, r, seed=1200 + M + K, dtype="bf16")
    want = gu.forward(p, "bf16", flags=stl.STL_FLAG_FUSED if single else stl.STL_FLAG_UNFUSED)
    assert np.array_equal(gu.forward(p, "bf16", flags=stl.STL_FLAG_AUTO), want)


@pytest.mark.parametrize("M,K,N,r,single", [(64, 48, 64, 32, False), (128, 48, 128, 32, False), (224, 32, 256, 25, False), (256, 48, 256, 32, True),
                                            (128, 16, 160, 32, True), (128, 48, 128, 24, True), (32, 48, 64, 32, True)])
def test_automatic_choice_that_saves_yhat(gu, M, K, N, r, single):
    """The store of Yhat costs the single launch more than the three: few blocks of more than 24 planes stay with those."""
    import paper_2503_12211_amd as stl
    p = stl_synth.stl_problem(4 * M, 4 * K, 4 * N, r, seed=1250 + M + K + r, dtype="bf16")
    want = gu.forward(p, "bf16", flags=stl.STL_FLAG_FUSED if single else stl.STL_FLAG_UNFUSED, save_yhat=True)
    other = gu.forward(p, "bf16", flags=stl.STL_FLAG_UNFUSED if single else stl.STL_FLAG_FUSED, save_yhat=True)
    got = gu.forward(p, "bf16", flags=stl.STL_FLAG_AUTO, save_yhat=True)
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
    assert not np.array_equal(other[0], want[0])


@pytest.mark.parametrize("K,r", [(16, 8), (48, 3), (80, 16), (32, 9)])
def test_more_blocks_than_cus(gu, K, r):
    """288 blocks of 32 x 32 tiles, beyond one per CU: the oracle's values and, bit for bit, those of calls of 28 tile rows each, whose blocks
    have a CU each and a deeper ring of stages."""
    import paper_2503_12211_amd as stl
    p = stl_synth.stl_problem(4 * 1020, 4 * K, 4 * 288, r, seed=1300 + K + r, dtype="bf16")
    C = planes.forward(p["X"], p["What"], p["E_X"], p["D"])
    for flag in (stl.STL_FLAG_FUSED, stl.STL_FLAG_EPILOGUE):
        got = gu.forward(p, "bf16", flags=flag)
        gu.check(got, C, "bf16", "C")
        for row in (0, 512, 3968):
            few = dict(p, X=np.ascontiguousarray(p["X"][row:row + 112]))
            assert np.array_equal(gu.forward(few, "bf16", flags=flag), got[row:row + 112]), (flag, row)
