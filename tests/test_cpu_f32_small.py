"""Address check of the fp32 kernels for small matrices at the shapes of test_gpu_f32_small.py (see test_cpu_address_check.py)."""
from test_cpu_address_check import checker, pytestmark  # noqa: F401
from test_cpu_routes import desc


def test_blocks_by_shape(checker):  # noqa: F811
    """Shapes on either side of the rules, and those that test_gpu_f32_small.py runs on 64 x 64 blocks."""
    f32 = [(("Yhat", 64, 64, 64, 49), 32), (("Yhat", 300, 300, 300, 32), 32), (("Yhat", 256, 16, 256, 32), 64), (("dXhat", 256, 256, 16, 32), 64),
           (("Yhat", 256, 32, 256, 32), 64), (("Yhat", 256, 33, 256, 32), 32), (("Yhat", 250, 32, 254, 40), 64), (("Yhat", 250, 32, 254, 3), 32), (("Yhat", 512, 512, 512, 32), 128), (("Yhat", 384, 384, 384, 56), 32),
           (("Yhat", 250, 9, 254, 40), 64), (("dXhat", 250, 254, 9, 40), 64), (("dWhat", 17, 254, 190, 64), 64)]
    bf16 = [(("dXhat", 256, 256, 7, 40), 64), (("dXhat", 1000, 64, 6, 32), 64), (("dWhat", 7, 512, 512, 8), 64), (("dWhat", 3, 128, 128, 16), 32),
            (("dWhat", 4, 512, 512, 32), 128), (("Yhat", 250, 7, 254, 40), 64), (("dXhat", 250, 254, 7, 40), 64), (("dWhat", 5, 250, 254, 40), 64)]
    stacked = [((126, 126, 12, 64, 0, 1, 0, 64, 64, 64, 2), 64), ((120, 126, 12, 48, 0, 0, 0, 64, 64, 64, 3), 64), ((126, 126, 12, 64, 1, 1, 0, 64, 64, 64, 2), 64)]
    args = ["f32,route:" + ":".join(map(str, desc(*c))) for c, _ in f32] + ["route:" + ":".join(map(str, desc(*c))) for c, _ in bf16]
    args += ["f32,route:" + ":".join(map(str, d)) for d, _ in stacked]
    _, text = checker(*args)
    got = [tuple(ln.split()[1:]) for ln in text.splitlines() if ln.startswith("  route")]
    assert got == [("generic", f"{b}x{b}") for _, b in f32 + bf16 + stacked]


def test_f32_small_addresses(checker):  # noqa: F811
    checker("f32,bwd:16:256:256:16", "f32,bwd:20:252:260:17", "f32,bwd:132:12:520:33", "f32,bwd:280:128:36:48", "f32,bwd:256:260:4:49",
            "f32,bwd:124:512:132:64", "f32,bwd:800:1000:24:3", "f32,bwd:4120:64:160:8", "f32,bwd:772:1028:256:40", "f32,bwd:4092:264:280:64",
            "f32,ewb:256:256:49", "f32,ragged:9:39:36:60:49", "f32,ragged:3:198:64:96:24", "f32,aa:3:36:36:44:8", "bwd:28:4096:4096:32",
            "f32,bwd:2048:2048:2048:32", "f32,bwd:1000:36:1016:40", "f32,bwd:1000:1016:36:40", "f32,bwd:68:1016:760:64", "bwd:1000:28:1016:40",
            "bwd:1000:1016:28:40", "bwd:20:1000:1016:40", "f32,aa:2:504:48:504:64", "f32,aa:3:480:504:48:48", "f32,aa:2:48:504:504:64")
