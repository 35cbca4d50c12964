"""Automatic choice of the forward variant: the single-launch variant's bits wherever the rule takes it, and right against the
oracle on either side of the rule's edges at r <= 8 (128 tile columns of X and 256 blocks of 32 x 32 tiles) and of 4.2 million tile
products at any contraction length and rank.  The edges at r <= 16 (112 tile columns), r <= 32 (48) and with Yhat saved are in
test_gpu_single_launch.py."""
import numpy as np
import pytest

import stl_synth
from oracle import planes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gu():
    import gpu_util
    return gpu_util


@pytest.mark.parametrize("m,k,n,r,single", [(1024, 512, 512, 8, True), (4096, 256, 1024, 5, True), (4100, 512, 992, 8, False),
                                            (1024, 576, 512, 8, False), (1024, 512, 512, 9, False), (1020, 448, 1056, 7, True),
                                            (32, 1024, 512, 8, True), (32, 2048, 512, 8, True), (32, 2048, 544, 8, False),
                                            (128, 256, 256, 32, True), (132, 256, 256, 32, False)])
def test_auto_forward(gu, m, k, n, r, single):
    import paper_2503_12211_amd as stl
    p = stl_synth.stl_problem(m, k, n, r, seed=600 + m + k + n + r, dtype="bf16")
    got = gu.forward(p, "bf16")
    gu.check(got, planes.forward(p["X"], p["What"], p["E_X"], p["D"]), "bf16", "C")
    flag = stl.STL_FLAG_FUSED if single else stl.STL_FLAG_UNFUSED
    assert np.array_equal(got, gu.forward(p, "bf16", flags=flag))
