"""Address check of the plane products of few rows at the shapes of test_gpu_few_rows.py (see test_cpu_address_check.py)."""
from test_cpu_address_check import checker, pytestmark  # noqa: F401


def test_few_rows_addresses(checker):  # noqa: F811
    checker("bwd:32:32:64:3", "bwd:32:32:32:1", "bwd:64:1056:544:49", "bwd:36:4000:992:8", "bwd:60:1184:4064:64", "bwd:4:3104:224:40", "bwd:28:4000:992:8",
            "bwd:128:512:512:5", "bwd:68:544:4128:9", "bwd:124:2080:4096:32", "bwd:68:8192:224:4", "bwd:132:512:512:5", "bwd:64:4096:4096:32",
            "bwd:128:512:4096:32", "bwd:68:640:4128:17",
            "aa:1:64:256:288:9", "aa:1:20:160:1056:33")
