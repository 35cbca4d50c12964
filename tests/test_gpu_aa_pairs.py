"""Two activations: both operands encoded by one launch, and the backward that decodes both gradients by one launch and adds up three sums by
one (everything saved and everything asked for) against the calls that take the steps one by one (nothing saved, so everything is
recomputed): the same kernels' arithmetic in the same order, bit for bit; and the forward against the oracle.  Widths of 8 to 32
tiles share items of several tile rows, incomplete ones at the end of the stack and of a row included.

Bars: gpu_util.check (see test_gpu_any_width.py)."""
import numpy as np
import pytest

import stl_synth
from oracle import planes

pytestmark = pytest.mark.gpu

OUTS = ("dA", "dB", "dE_A", "dE_B", "dD")


@pytest.fixture(scope="module")
def gu():
    import gpu_util
    return gpu_util


@pytest.mark.parametrize("nb,M,K,N,r,bt", [(9, 50, 16, 50, 32, True), (3, 33, 8, 9, 17, True), (2, 67, 20, 64, 49, False), (5, 13, 32, 31, 8, True),
                                           (4, 65, 66, 8, 64, False), (1, 9, 11, 30, 5, True), (7, 30, 33, 17, 24, False), (3, 128, 24, 128, 40, True)])
def test_pairs(gu, nb, M, K, N, r, bt):
    import torch

    import paper_2503_12211_amd as stl
    fl = stl.STL_FLAG_B_TRANSPOSED if bt else 0
    p = stl_synth.aa_problem(nb, 4 * M, 4 * K, 4 * N, r, seed=1300 + M + K + N + r, dtype="bf16", with_dC=True)
    B = p["B"]
    if bt:
        B = np.ascontiguousarray(np.concatenate([B[b * 4 * K:(b + 1) * 4 * K].T for b in range(nb)], axis=0))
    prob = stl.Problem(4 * M, 4 * K, 4 * N, r)
    A, Bd, E_A, E_B, D, dC = (gu.dev(x, "bf16") for x in (p["A"], B, p["E_A"], p["E_B"], p["D"], p["dC"]))
    RB, CB = (nb * N, K) if bt else (nb * K, N)

    def buf(rows, cols):
        return torch.full((stl.stl_plane_elems(rows, cols, r),), float("nan"), dtype=torch.bfloat16, device="cuda")

    saved = [buf(nb * M, K), buf(RB, CB), buf(nb * M, N)]
    C = torch.empty((4 * nb * M, 4 * N), dtype=torch.bfloat16, device="cuda")
    nf, nw = (stl.stl_aa_workspace_bytes(prob, nb, op) for op in (stl.STL_OP_FORWARD, stl.STL_OP_BACKWARD))
    stl.stl_aa_forward(prob, nb, A, Bd, E_A, E_B, D, C, *saved, torch.empty(nf, dtype=torch.uint8, device="cuda"), nf, fl)
    args = (p["A"], B, p["E_A"], p["E_B"], p["D"])
    gu.check(gu.host(C), planes.aa_forward(*args, nbatch=nb, b_transposed=bt), "bf16", "C")
    got = []
    for planes_in in (saved, [None] * 3):
        out = {"dA": torch.empty_like(A), "dB": torch.empty_like(Bd)}
        out.update({g: torch.full((r, 16), 2.0, device="cuda") for g in OUTS[2:]})
        ws = torch.full((nw + 256,), 0x55, dtype=torch.uint8, device="cuda")
        for acc in (0, 1):
            stl.stl_aa_backward(prob, nb, A, Bd, E_A, E_B, D, dC, *planes_in, *(out[o] for o in OUTS), acc, ws, nw, fl)
        assert bool((ws[nw:] == 0x55).all())
        got.append(out)
    ref = dict(zip(OUTS, planes.aa_backward(*args, p["dC"], nbatch=nb, b_transposed=bt)))
    for o in OUTS:
        assert torch.equal(got[0][o], got[1][o]), o
        assert gu.rel(gu.host(got[0][o]) / (2 if o.startswith(("dE", "dD")) else 1), ref[o]) <= gu.TOL["bf16"], o
