"""Address check of the bf16 kernels at tile counts that are no multiple of 8 (see test_cpu_address_check.py)."""
from test_cpu_address_check import checker, pytestmark  # noqa: F401


def test_any_width_addresses(checker):  # noqa: F811
    checker("bwd:36:32:36:32", "bwd:32:60:32:5", "bwd:132:252:260:17", "bwd:260:36:508:49", "bwd:516:516:264:24",
            "bwd:2048:768:1000:32", "bwd:1200:260:4004:16", "bwd:64:28:36:8", "bwd:28:48:40:8",
            "mlp:64:36:1000:24", "mlp:36:264:260:49", "ewb:1000:36:24", "ewb:36:1000:49", "aa:4:200:64:200:32", "aa:3:36:36:44:8",
            "ragged:3:197:100:1000:32", "ragged:2:39:36:60:49")
