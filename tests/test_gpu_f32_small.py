"""fp32 steps of small matrices: the basis gradients shared by several workgroups per partial (tile_grad_kernel) and the plane products of
32 x 32 and 64 x 64 blocks, at the edges of partials (256 tiles), of planes per workgroup (16), of narrow rows (several tile rows per item), of
blocks (32) and of contraction stages (64), and on either side of the rules that choose them.

Bars: gpu_util.check, relative Frobenius error 1e-5 and every entry within 5e-5 rms (fp32)."""
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


@pytest.mark.parametrize("M,K,N,r", [(4, 64, 64, 16), (5, 63, 65, 17), (33, 3, 130, 33), (70, 32, 9, 48), (64, 65, 1, 49), (31, 128, 33, 64),
                                     (200, 250, 6, 3), (1030, 16, 40, 8), (193, 257, 64, 40), (1023, 66, 70, 64)])
def test_step_f32_small(gu, M, K, N, r):
    p = stl_synth.stl_problem(4 * M, 4 * K, 4 * N, r, seed=600 + M + K + N + r, dtype="f32", with_dC=True)
    got = gu.step(p, "f32")
    C, Y = planes.forward(p["X"], p["What"], p["E_X"], p["D"], return_yhat=True)
    gu.check(got["C"], C, "f32", "C")
    gu.check(got["Yhat"], Y, "f32", "Yhat", slab=1)
    ref = dict(zip(NAMES, planes.backward(p["X"], p["What"], p["E_X"], p["D"], p["dC"])))
    for name in NAMES:
        gu.check(got[name], ref[name], "f32", name)
    init = [np.ones_like(ref[nm], dtype=np.float32) for nm in NAMES[1:]]
    acc = gu.backward(p, "f32", accumulate=1, init=init)
    for nm in NAMES[1:]:
        # one rounding of (1 + gradient) on top of the same sums
        assert np.abs(acc[nm] - 1.0 - got[nm]).max() <= 2.0 ** -22 * max(1.0, np.abs(got[nm]).max()), nm
    alone = gu.backward(p, "f32", skip=("dX", "dWhat"))
    for nm in ("dE_X", "dD"):
        assert gu.rel(alone[nm], ref[nm]) <= gu.TOL["f32"], nm


def check_products(gu, p, dtype):
    got = gu.step(p, dtype)
    C, Y = planes.forward(p["X"], p["What"], p["E_X"], p["D"], return_yhat=True)
    gu.check(got["Yhat"], Y, dtype, "Yhat", slab=1)
    gu.check(got["C"], C, dtype, "C")
    ref = dict(zip(NAMES, planes.backward(p["X"], p["What"], p["E_X"], p["D"], p["dC"])))
    for name in NAMES:
        gu.check(got[name], ref[name], dtype, name)
    acc = gu.backward(p, dtype, accumulate=1, init=[np.ones_like(ref[nm], dtype=np.float32) for nm in NAMES[1:]])
    assert np.abs(acc["dWhat"] - 1.0 - got["dWhat"]).max() <= 2.0 ** -22 * max(1.0, np.abs(got["dWhat"]).max())


@pytest.mark.parametrize("dtype,M,K,N,r", [("f32", 250, 9, 254, 40), ("f32", 250, 254, 9, 40), ("f32", 17, 254, 190, 64), ("bf16", 250, 7, 254, 40),
                                           ("bf16", 250, 254, 7, 40), ("bf16", 5, 250, 254, 40)])
def test_blocks_of_64(gu, dtype, M, K, N, r):
    """Contractions of one stage of 32 over incomplete blocks: the forward product, the input gradient's and the weight gradient's in turn."""
    check_products(gu, stl_synth.stl_problem(4 * M, 4 * K, 4 * N, r, seed=640 + M + K + N + r, dtype=dtype, with_dC=True), dtype)


@pytest.mark.parametrize("nb,M,K,N,r", [(2, 126, 12, 126, 64), (3, 120, 126, 12, 48), (2, 12, 126, 126, 64)])
def test_stacked_blocks_of_64(gu, nb, M, K, N, r):
    p = stl_synth.aa_problem(nb, 4 * M, 4 * K, 4 * N, r, seed=660 + M + K + N, dtype="f32", with_dC=True)
    args = (p["A"], p["B"], p["E_A"], p["E_B"], p["D"])
    gu.check(gu.aa_forward(*args, nb, "f32"), planes.aa_forward(*args, nbatch=nb), "f32", "C")
    got = gu.aa_backward(*args, p["dC"], nb, "f32")
    for name, ref in zip(("dA", "dB", "dE_A", "dE_B", "dD"), planes.aa_backward(*args, p["dC"], nbatch=nb)):
        gu.check(got[name], ref, "f32", name)


@pytest.mark.parametrize("dtype,M,K,N,r", [("f32", 250, 9, 254, 40), ("f32", 250, 32, 254, 40), ("bf16", 250, 7, 254, 40)])
def test_blocks_of_64_add_up_as_blocks_of_32_do(gu, dtype, M, K, N, r):
    """The same products with fewer planes, which take 32 x 32 blocks: bit for bit."""
    p = stl_synth.stl_problem(4 * M, 4 * K, 4 * N, r, seed=680 + K, dtype=dtype)
    _, Y = gu.forward(p, dtype, flags=1, save_yhat=True)
    few = dict(p, **{s: np.ascontiguousarray(p[s][:3]) for s in ("What", "E_X", "D")})
    assert np.array_equal(Y[:3], gu.forward(few, dtype, flags=1, save_yhat=True)[1])
