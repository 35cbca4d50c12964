"""The tile maps and plane products of fp32 storage (and of bf16 planes with a dimension below 8) at the edges of their items
(64 tiles, narrow matrices packed several tile rows to an item), plane groups (16), stages (16 and 32) and blocks (64, 128).

Bars as everywhere: gpu_util.check, 1e-5 relative and 5e-5 rms per entry for fp32 (sums of at most a few thousand fp32 terms:
2^-24 sqrt(terms) is below 4e-6), 1e-2 / 0.05 for bf16."""
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


SHAPES = [("f32", 1, 1, 1, 1), ("f32", 3, 5, 2, 16), ("f32", 64, 64, 64, 49), ("f32", 65, 63, 33, 17), ("f32", 17, 130, 66, 64),
          ("f32", 300, 4, 129, 33), ("f32", 129, 200, 130, 48), ("f32", 513, 31, 8, 2), ("f32", 260, 97, 257, 32),
          ("bf16", 5, 7, 3, 16), ("bf16", 40, 2, 70, 49), ("bf16", 6, 64, 5, 33)]


@pytest.mark.parametrize("dtype,M,K,N,r", SHAPES)
def test_step_edges(gu, dtype, M, K, N, r):
    p = stl_synth.stl_problem(4 * M, 4 * K, 4 * N, r, seed=500 + M + K + N + r, dtype=dtype, with_dC=True)
    got = gu.step(p, dtype)
    C, Y = planes.forward(p["X"], p["What"], p["E_X"], p["D"], return_yhat=True)
    gu.check(got["C"], C, dtype, "C")
    gu.check(got["Yhat"], Y, dtype, "Yhat", slab=1)
    ref = dict(zip(NAMES, planes.backward(p["X"], p["What"], p["E_X"], p["D"], p["dC"])))
    for name in NAMES:
        gu.check(got[name], ref[name], dtype, name)
    init = [np.ones_like(ref[nm], dtype=np.float32) for nm in NAMES[1:]]
    acc = gu.backward(p, dtype, accumulate=1, init=init)
    for nm in NAMES[1:]:
        # one rounding of (1 + gradient) on top: 2^-24 of the larger of the two
        assert np.abs(acc[nm] - 1.0 - got[nm]).max() <= 2.0 ** -22 * max(1.0, np.abs(got[nm]).max()), nm
    alone = gu.backward(p, dtype, skip=("dX", "dWhat"))
    for nm in ("dE_X", "dD"):
        assert np.array_equal(alone[nm], got[nm]), nm
