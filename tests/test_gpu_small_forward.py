"""The single-launch forward on 16 x 16 tiles: incomplete blocks in both directions, contractions of fewer steps than are in flight, of
exactly as many and of more, ending in half a step, ranks on either side of 8, 16 and 32 planes and of the four- and eight-plane groups of
its decodes; what it does not round equals the 32 x 32 blocks bit for bit (the decode-in-epilogue variant runs them, on the same rounded
Xhat), what it rounds three launches, on either side of the automatic choice's lines.

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


# M, K, N tile counts, r
SHAPES = [(1, 16, 8, 1), (17, 48, 24, 8), (33, 64, 40, 5), (16, 80, 16, 9), (31, 96, 48, 16), (48, 112, 72, 17), (15, 128, 136, 25), (260, 160, 232, 32),
          (64, 32, 2048, 16), (9, 208, 8, 31)]


@pytest.mark.parametrize("M,K,N,r", SHAPES)
def test_fused(gu, M, K, N, r):
    import paper_2503_12211_amd as stl
    p = stl_synth.stl_problem(4 * M, 4 * K, 4 * N, r, seed=1500 + M + K + N + r, dtype="bf16")
    C, Y = planes.forward(p["X"], p["What"], p["E_X"], p["D"], return_yhat=True)
    got, yhat = gu.forward(p, "bf16", flags=stl.STL_FLAG_FUSED, save_yhat=True)
    assert gu.rel(got, C) <= gu.TOL["bf16"] and gu.rel(yhat, Y) <= gu.TOL["bf16"]
    assert np.array_equal(gu.forward(p, "bf16", flags=stl.STL_FLAG_FUSED), got)
    blocks = gu.forward(p, "bf16", flags=stl.STL_FLAG_EPILOGUE, save_yhat=True)
    assert np.array_equal(got, blocks[0]) and np.array_equal(yhat, blocks[1])
    out = gu.forward(p, "bf16", flags=stl.STL_FLAG_FUSED | stl.STL_FLAG_GELU)
    assert gu.rel(out, planes.gelu(C)) <= gu.TOL["bf16"]


# the last contraction that one launch takes and the first that three do: the same bits either way
@pytest.mark.parametrize("M,K,N,r", [(256, 640, 256, 8), (256, 656, 256, 8), (250, 384, 256, 16), (256, 400, 248, 16), (256, 256, 256, 32), (256, 272, 256, 32),
                                     (512, 256, 256, 7), (512, 272, 256, 7), (500, 192, 256, 13), (500, 208, 256, 13), (34, 144, 264, 25), (513, 160, 256, 8)])
def test_rounded_is_three_launches(gu, M, K, N, r):
    import paper_2503_12211_amd as stl
    p = stl_synth.stl_problem(4 * M, 4 * K, 4 * N, r, seed=1600 + M + K + N + r, dtype="bf16")
    for flag in (0, stl.STL_FLAG_GELU):
        got, want = (gu.forward(p, "bf16", flags=f | flag, save_yhat=True) for f in (stl.STL_FLAG_AUTO, stl.STL_FLAG_UNFUSED))
        assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
        assert np.array_equal(gu.forward(p, "bf16", flags=stl.STL_FLAG_AUTO | flag), want[0])


@pytest.mark.parametrize("M,K,N,r,single", [(16, 256, 4096, 8, True), (16, 272, 1024, 8, False), (7, 256, 1024, 12, True), (20, 128, 1024, 32, True),
                                            (4, 144, 1024, 32, False)])
def test_few_rows(gu, M, K, N, r, single):
    """Up to 32 tile rows, whose three launches add up in another order."""
    import paper_2503_12211_amd as stl
    p = stl_synth.stl_problem(4 * M, 4 * K, 4 * N, r, seed=1700 + M + K + r, dtype="bf16")
    got = gu.forward(p, "bf16", flags=stl.STL_FLAG_AUTO)
    gu.check(got, planes.forward(p["X"], p["What"], p["E_X"], p["D"]), "bf16", "C")
    assert np.array_equal(got, gu.forward(p, "bf16", flags=stl.STL_FLAG_FUSED if single else stl.STL_FLAG_UNFUSED))


def test_infinities_stay_where_they_belong(gu):
    """An infinite entry of X reaches its own four rows of C, one of a weight plane its own four columns, also where both lie in the last,
    half step and beside rows and columns that a block does not have."""
    import paper_2503_12211_amd as stl
    p = stl_synth.stl_problem(4 * 40, 4 * 144, 4 * 136, 7, seed=1800, dtype="bf16")
    X, What = p["X"].copy(), p["What"].copy()
    X[4 * 39 + 1, 4 * 143] = np.inf
    What[6, 143, 135] = np.inf
    for flag in (stl.STL_FLAG_FUSED, stl.STL_FLAG_AUTO):
        clean = gu.forward(p, "bf16", flags=flag)
        got = gu.forward(dict(p, X=X, What=What), "bf16", flags=flag)
        assert np.isfinite(got[:4 * 39, :4 * 135]).all() and np.array_equal(got[:4 * 39, :4 * 135], clean[:4 * 39, :4 * 135])
        assert not np.isfinite(got[4 * 39:]).any() and not np.isfinite(got[:, 4 * 135:]).any()
