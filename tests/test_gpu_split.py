"""Plane products whose last, not full round of 256 x 256 blocks is dealt out in parts of 128 x 256 or 128 x 128: parts that hang over
the edge or do not exist, contractions of one pair of stages and of several rings, ending inside a stage (weight gradient); several parts
per workgroup: against the oracle, and bit for bit against the same planes a few at a time, which are whole blocks.  test_cpu_split.py
asserts which product of which shape is split.

Bars: gpu_util.check (see test_gpu_any_width.py)."""
import numpy as np
import pytest

import stl_synth
from oracle import planes

pytestmark = pytest.mark.gpu

NAMES = ("dX", "dWhat", "dE_X", "dD")

# M, K, N tile counts, r -> what becomes of the last round of Yhat, dXhat, dWhat, dWhat added to
SHAPES = {(648, 64, 264, 64): ("128x256", "whole", "whole", "whole"),
          (386, 128, 776, 40): ("128x128", "whole", "whole", "whole"),
          (648, 264, 64, 64): ("whole", "128x256", "whole", "whole"),
          (776, 392, 128, 40): ("whole", "128x128", "whole", "whole"),
          (8, 648, 264, 64): ("whole", "whole", "128x256", "whole"),
          (128, 512, 776, 40): ("whole", "whole", "128x128", "whole"),
          # (Contractions are 8 and up: an entry of few products is off by up to 2^-8 of their sizes, and of the 27 million sums of 8 that
          # 648 x 648, r = 64 has the largest products are some 25 times the root mean square of a product, sqrt(8) less of the sum's:
          # 2^-8 25 / sqrt(8) = 0.035 from one product alone, beyond the bar of 0.05 with the others.  104 of them: 0.010 each.)
          (104, 648, 648, 64): ("whole", "whole", "128x128", "128x128"),
          (201, 392, 520, 64): ("whole", "whole", "128x256", "128x256"),
          (192, 648, 392, 64): ("whole", "whole", "128x256", "128x256"),
          (128, 648, 392, 49): ("whole", "whole", "128x128", "128x128")}


@pytest.mark.parametrize("M,K,N,r", SHAPES)
def test_step_in_parts(M, K, N, r):
    import gpu_util as gu
    p = stl_synth.stl_problem(4 * M, 4 * K, 4 * N, r, seed=900 + M + K + N + r, dtype="bf16", with_dC=True)
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


FEW = 8                  # planes of a product that is not cut (test_cpu_split.py)


@pytest.mark.parametrize("M,K,N,r", SHAPES)
def test_parts_add_up_like_whole_blocks(M, K, N, r):
    import torch

    import gpu_util as gu
    import paper_2503_12211_amd as stl
    yhat, dxhat, dwhat, dwhat_added = (x != "whole" for x in SHAPES[M, K, N, r])
    p = stl_synth.stl_problem(4 * M, 4 * K, 4 * N, r, seed=1000 + M + K + N + r, dtype="bf16", with_dC=True)
    rng = np.random.default_rng(M + K + N + r)
    Xh, Yh = (stl_synth.round_to(rng.standard_normal((r, M, Cc)), "bf16") for Cc in (K, N))
    few = [slice(a, min(a + FEW, r)) for a in range(0, r, FEW)]

    def part(c, **more):
        return dict(p, What=p["What"][c], E_X=p["E_X"][c], D=p["D"][c], **more)

    if yhat:
        def products(c):
            n = len(range(*c.indices(r)))
            Y = gu.planes_buffer(n, M, N, "bf16")
            stl.stl_plane_matmul(stl.Problem(4 * M, 4 * K, 4 * N, n), gu.planes_to_dev(Xh[c], "bf16"), gu.dev(p["What"][c], "bf16"), Y)
            torch.cuda.synchronize()
            return gu.planes_to_host(Y, n, M, N)
        got = products(slice(0, r))
        assert all(np.array_equal(got[c], products(c)) for c in few)
    init = [np.ones((r, K, N), dtype=np.float32), np.ones((r, 16), dtype=np.float32), np.ones((r, 16), dtype=np.float32)]
    for split, kw in ((dwhat, False), (dwhat_added, True)):
        if split:
            def gradient(q, c):
                more = {"accumulate": 1, "init": [x[c] for x in init]} if kw else {}
                return gu.backward(q, "bf16", yhat=Yh[c], xhat=Xh[c], skip=("dX", "dE_X", "dD"), **more)["dWhat"]
            got = gradient(p, slice(0, r))
            assert all(np.array_equal(got[c], gradient(part(c), c)) for c in few)
    if dxhat:
        def gradients(q, c):
            """dXhat: with a basis of unit vectors the entries of dX are planes of it."""
            n = q["What"].shape[0]
            out = []
            for a in range(0, n, 16):
                E = np.zeros((n, 16), dtype=np.float32)
                E[np.arange(a, min(a + 16, n)), np.arange(min(16, n - a))] = 1.0
                dX = gu.backward(dict(q, E_X=E), "bf16", yhat=Yh[c], xhat=Xh[c], skip=("dWhat", "dE_X", "dD"))["dX"]
                tiles = dX.reshape(M, 4, K, 4).transpose(1, 3, 0, 2).reshape(16, M, K)
                out.append(tiles[:min(16, n - a)])
            return np.concatenate(out)
        got = gradients(p, slice(0, r))
        assert all(np.array_equal(got[c], gradients(part(c), c)) for c in few)
