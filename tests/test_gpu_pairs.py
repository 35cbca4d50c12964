"""Gradients whose two plane products run as one launch, at sizes where one product has a single block, a single stage or an incomplete one,
or many more blocks than the other: against the oracle, and against calls that ask for one gradient at a time and so launch them apart,
bit for bit unless groups of wavefronts share a contraction there.  test_cpu_pairs.py asserts which run together, and which those are.

Bars: gpu_util.check (see test_gpu_any_width.py)."""
import numpy as np
import pytest

import stl_synth
import test_gpu_any_width
import test_gpu_blocks
import test_gpu_split
import test_gpu_staged
from oracle import planes

pytestmark = pytest.mark.gpu

NAMES = ("dX", "dWhat", "dE_X", "dD")

# dtype, M, K, N tile counts, r -> whether dWhat and dXhat run together
SHAPES = {("bf16", 9, 10, 11, 3): True, ("bf16", 64, 61, 63, 8): True, ("bf16", 65, 66, 67, 5): True, ("bf16", 50, 33, 130, 32): True,
          ("bf16", 130, 129, 20, 9): True, ("bf16", 12, 140, 951, 40): False, ("bf16", 15, 601, 479, 49): False, ("bf16", 130, 264, 70, 3): True,
          # contractions that two and four groups of wavefronts share where a product runs by itself
          ("bf16", 704, 67, 70, 3): True, ("bf16", 705, 67, 70, 3): False, ("bf16", 2899, 9, 195, 3): False, ("bf16", 70, 67, 706, 3): False,
          # widths that are multiples of 8: edges of 64 and 64, 64 and 128, 128 and 64, 128 and 128; contractions of part of a stage, of one, of as
          # many as a ring holds and of more
          ("bf16", 8, 16, 8, 3): True, ("bf16", 64, 64, 64, 5): True, ("bf16", 65, 136, 264, 9): True, ("bf16", 257, 72, 32, 33): True,
          ("bf16", 200, 128, 1000, 24): True, ("bf16", 200, 520, 512, 48): True, ("bf16", 526, 576, 576, 16): True, ("bf16", 1100, 80, 616, 16): True,
          ("bf16", 8, 1024, 264, 40): True, ("bf16", 1024, 1024, 1024, 32): False,
          ("f32", 1, 1, 1, 1): True, ("f32", 33, 31, 65, 7): True, ("f32", 64, 64, 64, 49): True, ("f32", 5, 130, 70, 16): True,
          ("f32", 100, 16, 30, 64): True}
# those of which a product's contraction is shared by groups of wavefronts where it runs by itself: sums in another order
SHARED = {("bf16", 704, 67, 70, 3)}
# nbatch, M, K, N, r, second operand stored transposed -> whether dAhat and dBhat do
AA_SHAPES = {(3, 9, 11, 13, 4, False): True, (3, 9, 11, 13, 4, True): True, (8, 50, 16, 50, 32, True): True, (8, 50, 50, 16, 32, False): True,
             (5, 70, 33, 66, 8, True): True, (5, 70, 66, 33, 8, False): True, (17, 100, 70, 20, 32, False): False,
             (2, 704, 67, 66, 3, False): True, (2, 705, 67, 66, 3, False): False, (1, 70, 66, 705, 5, True): False}
AA_SHARED = {(2, 704, 67, 66, 3, False)}


@pytest.fixture(scope="module")
def gu():
    import gpu_util
    return gpu_util


@pytest.mark.parametrize("dtype,M,K,N,r", SHAPES)
def test_layer(gu, dtype, M, K, N, r):
    p = stl_synth.stl_problem(4 * M, 4 * K, 4 * N, r, seed=1900 + M + K + N + r, dtype=dtype, with_dC=True)
    got = gu.step(p, dtype)
    ref = dict(zip(NAMES, planes.backward(p["X"], p["What"], p["E_X"], p["D"], p["dC"])))
    for name in NAMES:
        assert gu.rel(got[name], ref[name]) <= gu.TOL[dtype], name
    init = [np.ones_like(ref[nm], dtype=np.float32) for nm in NAMES[1:]]
    acc = gu.backward(p, dtype, accumulate=1, init=init)
    # one rounding of (1 + gradient) on top of the same sums
    assert np.abs(acc["dWhat"] - 1.0 - got["dWhat"]).max() <= 2.0 ** -22 * max(1.0, np.abs(got["dWhat"]).max())
    if (dtype, M, K, N, r) in SHARED:
        return
    # the same planes, dWhat without dXhat and dXhat without dWhat
    saved = {"xhat": got["Xhat"], "yhat": got["Yhat"]}
    alone = gu.backward(p, dtype, skip=("dWhat",), **saved)
    assert all(np.array_equal(alone[name], got[name]) for name in ("dX", "dE_X"))
    for kw in ({}, {"accumulate": 1, "init": init}):
        both, alone = (gu.backward(p, dtype, skip=skip, **saved, **kw)["dWhat"] for skip in ((), ("dX", "dE_X")))
        assert np.array_equal(both, alone)


@pytest.mark.parametrize("nb,M,K,N,r,bt", AA_SHAPES)
def test_pair_of_activations(gu, nb, M, K, N, r, bt):
    """The call that asks for everything against two that ask for one operand's gradients each."""
    import torch

    import paper_2503_12211_amd as stl
    m, k, n = 4 * M, 4 * K, 4 * N
    g = torch.Generator(device="cuda").manual_seed(2000 + nb + M + K + N)

    def normal(*shape, s=1.0):
        return (torch.randn(shape, generator=g, device="cuda") * s).to(torch.bfloat16)

    A, B, dC = normal(nb * m, k), normal(nb * (n if bt else k), k if bt else n, s=k ** -0.5), normal(nb * m, n)
    E_A, E_B, D = (normal(r, 16, s=0.25) for _ in range(3))
    prob, flags = stl.Problem(m, k, n, r, stl.STL_BF16), stl.STL_FLAG_B_TRANSPOSED if bt else 0
    ws_bytes = max(stl.stl_aa_workspace_bytes(prob, nb, op) for op in (stl.STL_OP_FORWARD, stl.STL_OP_BACKWARD))
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")

    def planes_of(R, Cc):
        return torch.empty(stl.stl_plane_elems(R, Cc, r), dtype=torch.bfloat16, device="cuda")

    Ah, Bh, Yh, C = planes_of(nb * M, K), planes_of(nb * N, K) if bt else planes_of(nb * K, N), planes_of(nb * M, N), torch.empty_like(dC)
    stl.stl_aa_forward(prob, nb, A, B, E_A, E_B, D, C, Ah, Bh, Yh, ws, ws_bytes, flags)

    def backward(a, b):
        out = {"dA": torch.empty_like(A) if a else None, "dB": torch.empty_like(B) if b else None}
        out.update({nm: torch.empty(r, 16, device="cuda") if want else None for nm, want in (("dE_A", a), ("dE_B", b), ("dD", a and b))})
        stl.stl_aa_backward(prob, nb, A, B, E_A, E_B, D, dC, Ah, Bh, Yh, out["dA"], out["dB"], out["dE_A"], out["dE_B"], out["dD"], 0, ws,
                            ws_bytes, flags)
        return out

    both, only_a, only_b = backward(True, True), backward(True, False), backward(False, True)
    for name, other in (("dA", only_a), ("dE_A", only_a), ("dB", only_b), ("dE_B", only_b)):
        x, y = both[name].double(), other[name].double()
        # basis gradients are added up in another order; so are the products if groups share a contraction (a rounding is turned over here and there)
        assert ((x - y).norm() / y.norm()).item() <= 1e-3, name
        assert name.startswith("dE") or (nb, M, K, N, r, bt) in AA_SHARED or torch.equal(x, y), name


ALONE = [*test_gpu_blocks.SHAPES, *test_gpu_split.SHAPES, *test_gpu_staged.SHAPES, *test_gpu_any_width.SHAPES]


@pytest.mark.parametrize("M,K,N,r", ALONE)
def test_gradients_on_their_own(gu, M, K, N, r):
    """The products of a call that asks for one gradient, over the shapes that reach every block, every last round in parts and every group of
    wavefronts."""
    p = stl_synth.stl_problem(4 * M, 4 * K, 4 * N, r, seed=2100 + M + K + N + r, dtype="bf16", with_dC=True)
    ref = dict(zip(NAMES, planes.backward(p["X"], p["What"], p["E_X"], p["D"], p["dC"])))
    gu.check(gu.backward(p, "bf16", skip=("dWhat", "dE_X", "dD"))["dX"], ref["dX"], "bf16", "dX")
    alone = ("dX", "dE_X", "dD")
    dW = gu.backward(p, "bf16", skip=alone)["dWhat"]
    gu.check(dW, ref["dWhat"], "bf16", "dWhat")
    init = [np.ones_like(ref[nm], dtype=np.float32) for nm in NAMES[1:]]
    acc = gu.backward(p, "bf16", accumulate=1, init=init, skip=alone)["dWhat"]
    # one rounding of (1 + gradient) on top of the same sums
    assert np.abs(acc - 1.0 - dW).max() <= 2.0 ** -22 * max(1.0, np.abs(dW).max())
