"""Which plane-product kernel a product takes: the host code's own rules, evaluated without a GPU (the driver of
test_cpu_address_check.py prints them)."""
from test_cpu_address_check import checker, pytestmark  # noqa: F401

from test_gpu_blocks import AA_SHAPES, SHAPES

PG = 64
BLOCKS = ("64x64", "128x128", "128x256", "256x256")


def desc(form, M, K, N, r):
    """The products of one layer as stl_api.hip describes them, tile counts: forward, input gradient, weight gradient (written,
    or added to what is there)."""
    return {"Yhat": (M, N, K, r, 0, 1, 0, PG, 0, PG, 1), "dXhat": (M, K, N, r, 0, 0, 0, PG, 0, PG, 1),
            "dWhat": (K, N, M, r, 1, 1, 1, PG, PG, 0, 1), "dWhat +=": (K, N, M, r, 1, 1, 2, PG, PG, 0, 1)}[form]


FORMS = ("Yhat", "dXhat", "dWhat", "dWhat +=")


def aa_descs(nb, M, K, N, r, bt):
    """The three products of stacked pairs of activations."""
    grads_b = (N, K, M) if bt else (K, N, M)
    return [(M, N, K, r, 0, 0 if bt else 1, 0, PG, PG, PG, nb), (M, K, N, r, 0, 1 if bt else 0, 0, PG, PG, PG, nb),
            grads_b + (r, 1, 1, 0, PG, PG, PG, nb)]


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
    assert routes(checker, [desc("dXhat", 2048, 1024, 131072, 64)]) == [("staged", "256x256")]


def test_large_fp32_tile_maps_go_one_tile_per_thread(checker):  # noqa: F811
    cases = {"f32,tiles:1:1024:1024:4": 1, "f32,tiles:1:2048:64:49": 1, "f32,tiles:0:16384:8:16": 1, "f32,tiles:0:2047:64:16": 0,
             "f32,tiles:1:64:64:49": 0, "f32,tiles:0:100000:7:16": 0, "tiles:1:16384:9:8": 1, "tiles:1:16384:9:9": 0,
             "tiles:1:16384:16:8": 0, "tiles:0:16384:9:8": 0, "tiles:1:16384:8:8": 0}
    _, text = checker(*cases)
    assert [int(ln.split()[1]) for ln in text.splitlines() if ln.startswith("  route")] == list(cases.values())


def test_large_fp32_tile_maps_addresses(checker):  # noqa: F811
    checker("f32,stages:1025:128:17", "f32,stages:16390:8:5", "f32,stages:2100:65:9", "f32,stages:130:1013:33", "stages:14570:9:8",
            "stages:8740:15:3", "f32,ragged:2800:197:32:36:5", "f32,ewb:520:4096:9")


def items(run, cases):
    """What the items of these encodes are: tile rows, tile columns, planes, rows of a group (activations 64, a weight all its rows),
    whether no row map lies between."""
    _, text = run(*("items:" + ":".join(map(str, c)) for c in cases))
    return [ln.split()[1] for ln in text.splitlines() if ln.startswith("  route")]


def test_items_of_bf16_encodes(checker):  # noqa: F811
    cases = {  # activations follow the planes where there are enough items, or few enough of them
             (8192, 508, 32, PG, 1): "flat", (4096, 1001, 49, PG, 1): "flat", (16384, 132, 49, PG, 1): "flat", (1024, 1004, 16, PG, 1): "flat",
             (3200, 200, 32, PG, 1): "flat", (2048, 1000, 32, PG, 1): "row", (8192, 512, 32, PG, 1): "row", (2049, 33, 8, PG, 1): "flat",
             (2048, 33, 8, PG, 1): "row",
             # a weight, and rows behind a row map: large planes of odd widths from a cache line on
             (8192, 508, 32, 8192, 1): "line_starts", (2001, 255, 64, 2001, 1): "line_starts", (8192, 508, 32, PG, 0): "line_starts",
             (2600, 250, 64, PG, 0): "line_starts", (8192, 512, 32, 8192, 1): "row", (16384, 132, 49, 16384, 1): "row", (1024, 1004, 16, 1024, 1): "row",
             # a weight of 64 tile rows is one group
             (64, 2100, 8, 64, 1): "flat", (63, 2100, 8, 63, 1): "row"}
    assert items(checker, cases) == list(cases.values())
    checker("stages:3401:193:49", "stages:2620:250:49", "stages:4001:252:33", "stages:1000:1001:32", "stages:527:2044:32", "stages:64:2100:8",
            "ragged:52:197:1000:32:64")


def test_encodes_of_few_narrow_rows_keep_items_of_a_row(checker):  # noqa: F811
    cases = {(1024, 15): "row", (1025, 15): "several_rows", (16, 9): "row", (4096, 32): "several_rows", (4096, 33): "flat", (4096, 7): "row"}
    assert items(checker, [(R, Cc, 16, PG, 1) for R, Cc in cases]) == list(cases.values())
    checker("stages:1024:9:49", "stages:1025:9:49", "stages:1027:31:17", "stages:1600:15:64", "stages:1030:16:33")


def test_block_forward_shares_a_cu_where_there_are_more_blocks(checker):  # noqa: F811
    """Up to a block per CU the ring of stages is as deep as LDS allows; beyond, two stages where several blocks then fit."""
    cases = {"ring:1:1024:256:8": 5, "ring:1:1024:257:8": 2, "ring:1:2048:1024:3": 2, "ring:0:1024:256:8": 5, "ring:0:1025:256:8": 2,
             "ring:0:1024:256:16": 4, "ring:0:2048:256:16": 2, "ring:1:1024:256:16": 3, "ring:1:2048:1024:16": 3, "ring:0:2048:256:17": 2,
             "ring:1:64:64:32": 2}
    _, text = checker(*cases)
    assert [int(ln.split()[1]) for ln in text.splitlines() if ln.startswith("  route")] == list(cases.values())
    # LDS and addresses of both rings, 256 and 288 blocks
    checker(*(f"fwd:4096:128:{n}:{r}:{v}" for n in (1024, 1152) for r in (5, 13) for v in (2, 3)))


def test_second_device_of_a_process(checker):  # noqa: F811
    """Dynamic LDS beyond 64 KB is granted per device and kernel: calls that ran on one device run on the next one too, and a kernel
    runs whether or not one of the same type ran before (the pipelined forward without and with GELU)."""
    cases = ("f32,bwd:64:32:48:49", "bwd:1024:512:512:32", "bwd:300:260:300:32", "fwd:64:64:64:32:3", "fwd:2048:256:1024:32:4",
             "fwd:2048:256:1024:32:260", "aa:2:256:128:256:32")
    checker(*cases, "device:1", *cases, "device:0", *cases)


def _covered(run, descs):
    """{(operand forms, fp32 output, stacked, kernel, block, ends inside a stage or any width)} that these products reach; 64 x 64 blocks
    staged through registers with the groups that share the contraction."""
    out = set()
    for d, (path, block) in zip(descs, routes(run, descs)):
        Mi, Nj, Kl, akm, bkm, f32, nb = d[0], d[1], d[2], d[4], d[5], d[6], d[10]
        odd = bool(Kl % 32) if path in ("rows", "wide", "pipe") else bool(Mi % 8 or Nj % 8 or Kl % 8)
        out.add((akm, bkm, f32, nb > 1, path, block, odd))
    return out


def _blocks(covered):
    """Without the groups of wavefronts, and without products of few rows, which have no such block."""
    return {k[:5] + (k[5].split(":")[0], k[6]) for k in covered if k[4] != "rows"}


def test_gpu_shapes_reach_every_kernel_form_and_block(checker):  # noqa: F811
    layer = _blocks(_covered(checker, [desc(f, *s) for s in SHAPES for f in FORMS]))
    forms = ((0, 1, 0), (0, 0, 0), (1, 1, 1), (1, 1, 2))
    want = {(a, b, f, False, "pipe", blk, tail) for a, b, f in forms for blk in BLOCKS for tail in (False, True)}
    want |= {(0, b, 0, False, "wide", "256x256", False) for b in (0, 1)}
    want |= {(a, b, f, False, "staged", blk, True) for a, b, f in forms for blk in ("64x64", "128x128", "256x256")}
    assert want - layer == set() and layer - want == set()
    aa = _blocks(_covered(checker, [d for s in AA_SHAPES for d in aa_descs(*s)]))
    want = {(1, 1, 0, False, "pipe", blk, tail) for blk in BLOCKS for tail in (False, True)}
    want |= {(1, 1, 0, False, "staged", blk, True) for blk in ("64x64", "128x128", "256x256")}
    for a, b in ((0, 1), (0, 0), (1, 1)):
        # stacked problems: the LDS-DMA kernel at one stage, otherwise staged
        want |= {(a, b, 0, True, "pipe", blk, False) for blk in BLOCKS}
        want |= {(a, b, 0, True, "staged", blk, odd) for blk in ("64x64", "128x128", "256x256") for odd in (False, True)}
    assert want - aa == set(), want - aa
    assert {k for k in aa if k[3]} - want == set()


def test_gpu_shapes_reach_every_group_of_wavefronts(checker):  # noqa: F811
    """64 x 64 blocks staged through registers: one stage, one group, two and four, for every operand form.  Two gradients of a layer may run as one
    launch, of one group: these shapes are also run one gradient at a time."""
    from test_gpu_any_width import SHAPES as ANY
    from test_gpu_pairs import ALONE
    from test_gpu_staged import SHAPES as STAGED, STACKED
    assert set(ANY + SHAPES + STAGED) <= set(ALONE)
    got = _covered(checker, [desc(f, *s) for s in ANY + SHAPES + STAGED for f in FORMS] + [d for s in AA_SHAPES + STACKED for d in aa_descs(*s)])
    got = {k[:3] + (k[5],) for k in got if k[4] == "staged" and ":" in k[5]}
    want = {form + (f"64x64:{g}",) for form in ((0, 1, 0), (0, 0, 0), (1, 1, 0), (1, 1, 1), (1, 1, 2)) for g in (0, 1, 2, 4)}
    assert want - got == set() and got - want == set()


def test_products_of_few_rows(checker):  # noqa: F811
    """Where the few-row kernel begins and ends, and that the shapes of test_gpu_few_rows.py reach all its forms."""
    from test_gpu_few_rows import OTHERS, SHAPES as FEW
    got = _covered(checker, [desc("Yhat", *s) for s in FEW])
    assert {k[4:] for k in got} == {("rows", f"{m}x{n}", tail) for m in (16, 32) for n in (64, 128) for tail in (False, True)}
    cases = {(16, 1024, 1024, 49): ("rows", "16x128"), (16, 1024, 1024, 16): ("rows", "16x64"), (3, 8, 8, 1): ("rows", "16x64"),
             (17, 128, 1024, 32): ("rows", "32x128"), (17, 120, 128, 5): ("pipe", "64x64"), (32, 512, 1024, 33): ("pipe", "64x64"),
             (33, 128, 128, 5): ("pipe", "64x64"), (16, 100, 96, 8): ("staged", "64x64:1"), (7, 100, 96, 8): ("generic", "32x32"), **{s: ("pipe", "64x64") for s in OTHERS}}
    assert routes(checker, [desc("Yhat", *s) for s in cases]) == list(cases.values())
    # the other products of the same layers stay where they are, and so do several stacked problems
    assert {p for p, _ in routes(checker, [desc(f, 16, 512, 512, 8) for f in FORMS[1:]])} == {"pipe"}
    assert {p for p, _ in routes(checker, aa_descs(2, 16, 512, 512, 8, False))} == {"staged"}


def test_blocks_that_were_measured_faster(checker):  # noqa: F811
    """Shapes on which the fastest block was at least 10 % ahead of the one taken by a rule without whole rounds and output types."""
    cases = {("Yhat", 1024, 256, 256, 49): "256x256", ("Yhat", 2048, 256, 256, 49): "256x256", ("Yhat", 1536, 512, 384, 16): "256x256",
             ("Yhat", 3200, 192, 768, 16): "256x256", ("dWhat", 2048, 256, 256, 49): "128x128",
             ("dWhat", 256, 512, 512, 49): "256x256", ("dWhat", 512, 768, 192, 49): "256x256", ("dWhat +=", 64, 256, 256, 8): "64x64"}
    got = routes(checker, [desc(*c) for c in cases])
    assert [block for _, block in got] == list(cases.values())


def test_listed_layers_of_the_any_width_tests(checker):  # noqa: F811
    """The shapes of test_gpu_any_width.py take the kernels they are meant for."""
    from test_gpu_any_width import SHAPES as ANY
    for s in ANY:
        want = "generic" if min(s[:3]) < 8 else "staged"
        assert {path for path, _ in routes(checker, [desc(f, *s) for f in FORMS])} == {want}, s
