"""bf16 encodes of large planes of odd widths, whose items follow the planes (activations, and a weight of one group) or begin on cache lines (other
weights, rows behind a row map): against the plane oracle, and bit for bit against the same rows encoded from a smaller matrix, whose
items begin with the row.  test_cpu_routes.py asserts which items they have."""
import numpy as np
import pytest

import stl_synth
from oracle import planes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gu():
    import gpu_util
    return gpu_util


def encode(gu, X, B, weight):
    import torch

    import paper_2503_12211_amd as stl
    (m, n), r = X.shape, B.shape[0]
    M, Cc = m // 4, n // 4
    gd = gu.Guard()
    if weight:
        P = gd.alloc((r, M, Cc), torch.bfloat16)
        stl.stl_encode_weight(stl.Problem(4, m, n, r), gu.dev(X, "bf16"), gu.dev(B, "bf16"), P)
        gd.check()
        return gu.host(P)
    P = gd.alloc((stl.stl_plane_elems(M, Cc, r),), torch.bfloat16)
    stl.stl_encode_activation(stl.Problem(m, n, n, r), gu.dev(X, "bf16"), gu.dev(B, "bf16"), P)
    gd.check()
    return gu.planes_to_host(P, r, M, Cc)


# widths: one more than three items, one less than four, multiple of 4, odd and large
@pytest.mark.parametrize("M,Cc,r,weight", [(3401, 193, 49, False), (2001, 255, 64, True), (4001, 252, 32, False), (1000, 1001, 33, False),
                                           (527, 2044, 32, True), (64, 2100, 8, True)])
def test_encode(gu, M, Cc, r, weight):
    rng = np.random.default_rng(M + Cc + r)
    X = stl_synth.round_to(rng.standard_normal((4 * M, 4 * Cc)), "bf16")
    B = stl_synth.round_to(rng.standard_normal((r, 16)) / 4, "bf16")
    P = encode(gu, X, B, weight)
    top = min(70, M - 1)
    assert np.array_equal(P[:, :top], encode(gu, X[:4 * top], B, weight))
    gu.check(P, planes.encode(X, B), "bf16", "planes", slab=1)


def test_ragged_rows(gu):
    """Through the row map: images of 197 rows, their null rows read as zeros."""
    p = stl_synth.ragged_problem(52, 197, 1000, 32, 64, seed=91, dtype="bf16")
    _, Xh, _ = gu.ragged_forward(p, 197, "bf16", save=True)
    gu.check(Xh, planes.encode(planes.pad_rows(p["X"], 197), p["E_X"]), "bf16", "Xhat", slab=1)
