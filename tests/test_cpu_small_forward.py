"""Addresses of the single-launch forward on 16 x 16 tiles (see test_cpu_address_check.py)."""
from test_cpu_address_check import checker, pytestmark  # noqa: F401

from test_gpu_small_forward import SHAPES


def test_small_forward_addresses(checker):  # noqa: F811
    # FUSED wherever it is taken, and the automatic choice
    checker(*(f"fwd:{4 * M}:{4 * K}:{4 * N}:{r}:{v}" for M, K, N, r in SHAPES if K % 16 == 0 and N % 8 == 0 for v in (3, 0)),
            "fwd:2048:1024:1024:7:0", "fwd:2000:768:1024:13:0", "fwd:136:576:1056:25:0")
