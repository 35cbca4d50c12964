"""Addresses of the tile maps whose items follow the planes (see test_cpu_address_check.py)."""
from test_cpu_address_check import checker, pytestmark  # noqa: F401

from test_gpu_flat_items import PAIRS, SHAPES


def test_flat_item_addresses(checker):  # noqa: F811
    checker(*(f"bwd:{4 * M}:{4 * K}:{4 * N}:{r}" for M, K, N, r in SHAPES), *(f"stages:{M}:{K}:{r}" for M, K, _, r in SHAPES), "stages:2100:100:32",
            "stages:520:1004:32", *("aa:" + ":".join(map(str, c)) for c in PAIRS), "aa:3:260:132:200:8", "aa:24:200:64:200:32", "mlp:260:148:264:16", "bwd:8200:400:400:16")
