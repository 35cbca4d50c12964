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
