"""Encodes and decodes that go one tile per thread (large fp32 matrices, and bf16 decodes of tall narrow ones at small ranks): against
the plane oracle at the edges of the rule (131072 tiles, 8 tile columns), of blocks (64 columns, 256, narrow ones), of the eight
planes in flight; and bit for bit against the kernel that a smaller matrix with the same rows takes (the sums run in the
same order).

Bars: gpu_util.check."""
import numpy as np
import pytest

import stl_synth
from oracle import planes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gu():
    import gpu_util
    return gpu_util


def stages(gu, dtype, X, B, gelu):
    """Planes of X, and the decode of those planes."""
    import torch

    import paper_2503_12211_amd as stl
    (m, n), r = X.shape, B.shape[0]
    M, Cc = m // 4, n // 4
    p = stl.Problem(m, n, n, r, gu.STL_DT[dtype])
    gd = gu.Guard()
    P, C = gd.alloc((stl.stl_plane_elems(M, Cc, r),), gu.TORCH_DT[dtype]), gd.alloc((m, n), gu.TORCH_DT[dtype])
    Bd = gu.dev(B, dtype)
    stl.stl_encode_activation(p, gu.dev(X, dtype), Bd, P)
    stl.stl_decode(p, P, Bd, C, stl.STL_FLAG_GELU if gelu else 0)
    gd.check()
    return gu.planes_to_host(P, r, M, Cc), gu.host(C)


@pytest.mark.parametrize("dtype,M,Cc,r,gelu", [("f32", 2048, 64, 49, False), ("f32", 1031, 128, 8, True), ("f32", 16384, 8, 7, False),
                                               ("f32", 14600, 9, 17, False), ("f32", 2048, 65, 64, False), ("f32", 130, 1013, 9, False),
                                               ("f32", 512, 257, 1, True), ("bf16", 14600, 9, 8, False), ("bf16", 8800, 15, 5, True)])
def test_against_the_oracle_and_the_item_kernels(gu, dtype, M, Cc, r, gelu):
    rng = np.random.default_rng(M + Cc + r)
    X = stl_synth.round_to(rng.standard_normal((4 * M, 4 * Cc)), dtype)
    B = stl_synth.round_to(rng.standard_normal((r, 16)) / 4, dtype)
    P, C = stages(gu, dtype, X, B, gelu)
    gu.check(P, planes.encode(X, B), dtype, "planes", slab=1)
    ref = planes.decode(P, B)
    gu.check(C, planes.gelu(ref) if gelu else ref, dtype, "matrix", entry_ref=ref)
    top = 64
    Pt, Ct = stages(gu, dtype, X[:4 * top], B, gelu)
    assert np.array_equal(P[:, :top], Pt)
    if dtype == "f32":                     # the bf16 decode of fewer tiles is the matrix cores', which add in another order
        assert np.array_equal(C[:4 * top], Ct)


@pytest.mark.parametrize("rows,K,N,r", [(197, 64, 65, 5), (39, 72, 96, 17)])
def test_ragged_rows(gu, rows, K, N, r):
    """Through the row map: null rows read as zeros and never written, the last tile rows decoded apart."""
    nimg = -(-140000 // ((rows // 4) * min(K, N)))
    p = stl_synth.ragged_problem(nimg, rows, 4 * K, 4 * N, r, seed=92, dtype="f32")
    C, Xh, Yh = gu.ragged_forward(p, rows, "f32", save=True)
    gu.check(Xh, planes.encode(planes.pad_rows(p["X"], rows), p["E_X"]), "f32", "Xhat", slab=1)
    gu.check(C, planes.ragged_forward(p["X"], p["What"], p["E_X"], p["D"], p["fold"], rows), "f32", "C")


def test_plane_major(gu):
    """The weight's layout: its encode, and dW alone from plane-major gradients."""
    import torch

    import paper_2503_12211_amd as stl
    K, N, r = 1031, 129, 9
    rng = np.random.default_rng(5)
    W = rng.standard_normal((4 * K, 4 * N)).astype(np.float32)
    E = (rng.standard_normal((r, 16)) / 4).astype(np.float32)
    dWh = rng.standard_normal((r, K, N)).astype(np.float32)
    gd = gu.Guard()
    What = gd.alloc((r, K, N), torch.float32)
    stl.stl_encode_weight(stl.Problem(4, 4 * K, 4 * N, r, stl.STL_F32), gu.dev(W, "f32"), gu.dev(E, "f32"), What)
    gd.check()
    gu.check(gu.host(What), planes.encode(W, E), "f32", "What", slab=1)
    got = gu.encode_weight_backward(W, E, dWh, "f32", skip=("dE_W",))
    gu.check(got["dW"], planes.encode_weight_backward(W, E, dWh)[0], "f32", "dW")
