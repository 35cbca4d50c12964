"""bf16 plane products over all their block sizes -- LDS-DMA kernels: 256 x 256, 128 x 256, 128 x 128, 64 x 64, whole-line form; products
staged through registers: 256 x 256, 128 x 128, 64 x 64 -- with blocks that hang over the edge and contractions that end inside a
stage of 32 (and, in the weight gradient, at any tile row).  test_cpu_routes.py asserts that the shapes below reach every
combination that exists.

Bars: gpu_util.check (see test_gpu_any_width.py)."""
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


# M, K, N tile counts, r -- blocks of the three products Yhat, dXhat, dWhat
SHAPES = [(16, 40, 64, 8),          # 64, 64, 64: fewer rows than a block
          (300, 200, 264, 3),       # 64, 64, 64
          (130, 72, 136, 49),       # 64, 64, 64
          (257, 488, 520, 40),      # 256, 128 x 256, 256; the weight gradient contracts over an odd number of rows
          (640, 320, 512, 24),      # 128 x 256, 128 x 256, 128 x 256
          (520, 264, 776, 32),      # 128, 128, 256
          (1030, 72, 520, 64),      # 128, 128, 128 x 256
          (2040, 232, 2040, 4),     # 256 with a contraction of 232; 64, 64
          # contractions of whole stages, more of them than a ring holds, beside some that end inside one
          (192, 160, 160, 3),       # 64, 64, 64
          (206, 160, 224, 49),      # 128, 128, 128
          (416, 264, 208, 48),      # 128 x 256, 256, 128
          (160, 832, 160, 40),      # 64, 256, 256
          (928, 160, 192, 33),      # 256, whole-line 256, 64
          (131, 192, 712, 48),      # whole-line 256, 64, 256
          # staged through registers, odd widths
          (100, 106, 111, 3),       # 64, 64, 64
          (305, 261, 134, 64),      # 128, 256, 128
          (288, 153, 271, 64),      # 256, 128, 128
          (128, 270, 265, 64)]      # 64, 64, 256

# stacked problems, M, K, N, r, second operand stored transposed -- the blocks that count
AA_SHAPES = [(1, 192, 160, 160, 3, False),        # one problem: the bf16 product of two [l][row] operands (dBhat) on
             (1, 154, 152, 152, 3, True),         #   64, with whole stages and without
             (1, 160, 672, 16, 49, False),        #   128
             (1, 164, 200, 216, 40, False),       #   128, ending inside a stage
             (1, 288, 480, 160, 64, False),       #   128 x 256
             (1, 208, 672, 16, 64, True),         #   128 x 256, ending inside a stage
             (1, 160, 400, 264, 64, False),       #   256
             (1, 421, 400, 272, 64, True),        #   256, ending inside a stage
             (1, 100, 106, 111, 3, False),        #   staged 64
             (1, 288, 153, 271, 64, True),        #   staged 128
             (1, 128, 270, 265, 64, False),       #   staged 256
             (2, 32, 32, 32, 3, False),           # stacked, one stage: 64, all three products
             (8, 80, 32, 16, 33, False),          #   128: Yhat
             (8, 16, 32, 80, 33, True),           #        Yhat with [j][l]
             (8, 32, 80, 16, 33, False),          #        dBhat
             (8, 144, 32, 16, 16, False),         #   128 x 256: Yhat
             (8, 144, 16, 32, 16, False),         #              dAhat
             (8, 32, 144, 16, 16, False),         #              dBhat
             (8, 272, 32, 144, 16, False),        #   256: Yhat
             (8, 288, 144, 32, 16, False),        #        dAhat
             (2, 32, 272, 144, 64, True),         #        dBhat
             (2, 80, 112, 80, 3, True),           # stacked, more stages: staged 128, multiples of 8
             (2, 160, 192, 160, 3, True),         #   staged 256, multiples of 8
             (2, 73, 75, 119, 3, True),           #   staged 64, odd widths
             (8, 77, 96, 93, 49, False),          #   staged 128
             (4, 194, 147, 145, 64, False)]       #   staged 256


@pytest.mark.parametrize("M,K,N,r", SHAPES)
def test_step_blocks(gu, M, K, N, r):
    p = stl_synth.stl_problem(4 * M, 4 * K, 4 * N, r, seed=700 + M + K + N + r, dtype="bf16", with_dC=True)
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


@pytest.mark.parametrize("nb,M,K,N,r,bt", AA_SHAPES)
def test_two_activation_blocks(gu, nb, M, K, N, r, bt):
    import paper_2503_12211_amd as stl
    FL = stl.STL_FLAG_B_TRANSPOSED if bt else 0
    p = stl_synth.aa_problem(nb, 4 * M, 4 * K, 4 * N, r, seed=900 + M + K + N + r, dtype="bf16", with_dC=True)
    B = p["B"]
    if bt:
        B = np.ascontiguousarray(np.concatenate([B[b * 4 * K:(b + 1) * 4 * K].T for b in range(nb)], axis=0))
    args = (p["A"], B, p["E_A"], p["E_B"], p["D"])
    gu.check(gu.aa_forward(*args, nb, "bf16", flags=FL), planes.aa_forward(*args, nbatch=nb, b_transposed=bt), "bf16", "C")
    got = gu.aa_backward(*args, p["dC"], nb, "bf16", flags=FL)
    ref = dict(zip(("dA", "dB", "dE_A", "dE_B", "dD"), planes.aa_backward(*args, p["dC"], nbatch=nb, b_transposed=bt)))
    for name in ref:
        gu.check(got[name], ref[name], "bf16", name)


@pytest.mark.parametrize("M,K,N,r", [(130, 72, 136, 9), (300, 40, 264, 5), (70, 250, 262, 4)])
def test_non_finite_rows_stay_where_they_are(gu, M, K, N, r):
    """Infinities and NaN in one tile row of X reach that tile row of C and no other: nothing of a neighbouring row enters a
    product."""
    p = stl_synth.stl_problem(4 * M, 4 * K, 4 * N, r, seed=800 + M, dtype="bf16")
    clean = gu.forward(p, "bf16")
    q = dict(p, X=p["X"].copy())
    row = M // 2
    q["X"][4 * row] = np.inf
    q["X"][4 * row + 1] = np.nan
    got = gu.forward(q, "bf16")
    others = np.r_[0:4 * row, 4 * row + 4:4 * M]
    assert np.array_equal(got[others], clean[others])
    assert not np.isfinite(got[4 * row:4 * row + 4]).all()


@pytest.mark.parametrize("dtype,M,K,N,r", [("bf16", 130, 72, 136, 9), ("bf16", 257, 488, 520, 40), ("bf16", 45, 272, 416, 64),
                                           ("bf16", 70, 250, 262, 4), ("bf16", 100, 130, 67, 3), ("f32", 50, 33, 70, 7)])
def test_weight_gradient_ends_with_the_rows(gu, dtype, M, K, N, r):
    """The weight gradient contracts over the tile rows: what lies behind them in the last group of a plane -- here NaN in the
    saved planes and in all of the workspace -- takes no part, not even multiplied by zero."""
    import torch

    import paper_2503_12211_amd as stl
    p = stl_synth.stl_problem(4 * M, 4 * K, 4 * N, r, seed=950 + M, dtype=dtype, with_dC=True)
    prob = stl.Problem(4 * M, 4 * K, 4 * N, r, gu.STL_DT[dtype])
    X, What, E_X, D, dC = (gu.dev(p[s], dtype) for s in ("X", "What", "E_X", "D", "dC"))
    nb = stl.stl_workspace_bytes(prob, stl.STL_OP_BACKWARD)
    got = []
    for fill in (0, 0xff):                                   # bytes 0xff: NaN in either type
        Xh, Y = (torch.full((stl.stl_plane_elems(M, w, r) * (4 if dtype == "f32" else 2),), fill, dtype=torch.uint8, device="cuda")
                 .view(gu.TORCH_DT[dtype]) for w in (K, N))
        ws = torch.full((nb,), fill, dtype=torch.uint8, device="cuda")
        stl.stl_forward(prob, X, What, E_X, D, torch.empty_like(dC), Xh, Y, ws, nb, stl.STL_FLAG_UNFUSED)
        assert bool(torch.isnan(Xh).any()) == bool(fill and M % gu.PG)         # the padding is untouched
        ws.fill_(fill)
        dWhat = torch.full((r, K, N), float("nan"), device="cuda")
        stl.stl_backward(prob, X, What, E_X, D, dC, Xh, Y, None, dWhat, None, None, 0, ws, nb)
        got.append(dWhat)
    assert bool(torch.isfinite(got[0]).all()) and torch.equal(got[0], got[1])
