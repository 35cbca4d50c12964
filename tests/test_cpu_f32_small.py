"""Address check of the fp32 kernels for small matrices at the shapes of test_gpu_f32_small.py (see test_cpu_address_check.py)."""
from test_cpu_address_check import checker, pytestmark  # noqa: F401


def test_f32_small_addresses(checker):  # noqa: F811
    checker("f32,bwd:16:256:256:16", "f32,bwd:20:252:260:17", "f32,bwd:132:12:520:33", "f32,bwd:280:128:36:48", "f32,bwd:256:260:4:49",
            "f32,bwd:124:512:132:64", "f32,bwd:800:1000:24:3", "f32,bwd:4120:64:160:8", "f32,bwd:772:1028:256:40", "f32,bwd:4092:264:280:64",
            "f32,ewb:256:256:49", "f32,ragged:9:39:36:60:49", "f32,ragged:3:198:64:96:24", "f32,aa:3:36:36:44:8", "bwd:28:4096:4096:32",
            "f32,bwd:2048:2048:2048:32")
