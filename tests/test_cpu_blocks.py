"""Address check of the plane products' block sizes and contraction tails (see test_cpu_address_check.py)."""
from test_cpu_address_check import checker, pytestmark  # noqa: F401


def test_block_addresses(checker):  # noqa: F811
    checker("bwd:64:160:256:8", "bwd:1200:800:1056:3", "bwd:520:288:544:49", "bwd:1028:1952:2080:40", "bwd:2560:1280:2048:24",
            "bwd:2080:1056:3104:32", "bwd:4120:288:2080:64", "bwd:8160:928:8160:4", "aa:4:128:128:256:8")
