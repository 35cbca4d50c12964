"""Which plane-product kernel a product takes: the host code's own rules, evaluated without a GPU (the driver of
test_cpu_address_check.py prints them)."""
from test_cpu_address_check import checker, pytestmark  # noqa: F401

PG = 64


def desc(form, M, K, N, r, nb=1):
    """The product descriptors of stl_api.hip, tile counts: the forward product Yhat, the input gradient dXhat and the weight
    gradient dWhat; `aa`: the same three of nb stacked pairs of activations (both operands and dBhat in the grouped layout)."""
    b = 0 if not form.startswith("aa_") else PG
    return {"Yhat": (M, N, K, r, 0, 1, 0, PG, b, PG, nb), "dXhat": (M, K, N, r, 0, 0, 0, PG, b, PG, nb),
            "dWhat": (K, N, M, r, 1, 1, 0 if b else 1, PG, PG, b, nb)}[form.removeprefix("aa_")]


def routes(run, descs):
    _, text = run(*("route:" + ":".join(map(str, d)) for d in descs))
    got = [tuple(ln.split()[1:]) for ln in text.splitlines() if ln.startswith("  route")]
    assert len(got) == len(descs)
    return got


def test_large_weights_stay_on_the_pipelined_kernels(checker):  # noqa: F811
    """A block reads at most 256 neighbouring rows of a plane-major weight, so its offsets fit 32 bits however many planes there
    are: the input gradients of layers of 16384 x 65536, 8192 x 151936 and, at r = 64, 32768 x 32768 run as smaller ones do."""
    shapes = [(2048, 4096, 16384, 32), (2048, 2048, 37984, 32), (2048, 8192, 8192, 64), (64, 4096, 16384, 49)]
    for (path, block), s in zip(routes(checker, [desc("dXhat", *s) for s in shapes]), shapes):
        assert path in ("wide", "pipe"), s
    # rows of a grouped operand lie further apart: here the offsets of 256 of them pass 32 bits and the product is staged
    # through registers
    assert routes(checker, [desc("dXhat", 2048, 1024, 131072, 64)]) == [("staged", "-")]


def test_large_fp32_tile_maps_go_one_tile_per_thread(checker):  # noqa: F811
    cases = {"f32,tiles:1:1024:1024:4": 1, "f32,tiles:1:2048:64:49": 1, "f32,tiles:0:16384:8:16": 1, "f32,tiles:0:2047:64:16": 0,
             "f32,tiles:1:64:64:49": 0, "f32,tiles:0:100000:7:16": 0, "tiles:1:16384:9:8": 1, "tiles:1:16384:9:9": 0,
             "tiles:1:16384:16:8": 0, "tiles:0:16384:9:8": 0, "tiles:1:16384:8:8": 0}
    _, text = checker(*cases)
    assert [int(ln.split()[1]) for ln in text.splitlines() if ln.startswith("  route")] == list(cases.values())


def test_large_fp32_tile_maps_addresses(checker):  # noqa: F811
    checker("f32,stages:1025:128:17", "f32,stages:16390:8:5", "f32,stages:2100:65:9", "f32,stages:130:1013:33", "stages:14570:9:8",
            "stages:8740:15:3", "f32,ragged:2800:197:32:36:5", "f32,ewb:520:4096:9")


def test_wide_bf16_encodes_of_odd_widths_write_whole_lines(checker):  # noqa: F811
    cases = {"lines:8192:508:32": 1, "lines:4096:1001:49": 1, "lines:8192:512:32": 0, "lines:16384:132:49": 0, "lines:1024:1004:16": 0}
    _, text = checker(*cases)
    assert [int(ln.split()[1]) for ln in text.splitlines() if ln.startswith("  route")] == list(cases.values())
    checker("stages:3401:193:49", "stages:2620:250:49", "stages:4001:252:33", "stages:1000:1001:32", "stages:527:2044:32", "ragged:52:197:1000:32:64")


def test_second_device_of_a_process(checker):  # noqa: F811
    """Dynamic LDS beyond 64 KB is granted per device and kernel: calls that ran on one device run on the next one too, and a kernel
    runs whether or not one of the same type ran before (the pipelined forward without and with GELU)."""
    cases = ("f32,bwd:64:32:48:49", "bwd:1024:512:512:32", "bwd:300:260:300:32", "fwd:64:64:64:32:3", "fwd:2048:256:1024:32:4",
             "fwd:2048:256:1024:32:260", "aa:2:256:128:256:32")
    checker(*cases, "device:1", *cases, "device:0", *cases)
