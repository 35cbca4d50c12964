"""Address check of the register-staged plane products at the shapes of test_gpu_staged.py (see test_cpu_address_check.py)."""
from test_cpu_address_check import checker, pytestmark  # noqa: F401


def test_staged_addresses(checker):  # noqa: F811
    checker("bwd:124:128:132:3", "bwd:252:256:260:2", "bwd:772:1028:36:5", "bwd:68:2820:3076:4", "bwd:2820:36:268:3", "bwd:3332:260:68:8",
            "bwd:280:772:516:49", "aa:9:200:64:200:8", "aa:5:132:36:124:49", "aa:3:256:64:256:32", "aa:3:192:256:96:5", "aa:2:1028:36:1284:8",
            "aa:96:200:64:200:32", "aa:1:2820:264:268:3", "aa:1:3332:268:260:3", "bwd:2048:768:1000:32")
