"""Gradients whose two plane products run as one launch: the rule, and addresses (see test_cpu_address_check.py)."""
from test_cpu_address_check import checker, pytestmark  # noqa: F401
from test_cpu_routes import aa_descs, desc, routes

from test_gpu_pairs import AA_SHAPES, AA_SHARED, SHAPES, SHARED


def paired(run, cases):
    _, text = run(*cases)
    return [int(ln.split()[1]) for ln in text.splitlines() if ln.startswith("  route")]


def name(dtype, *descs):
    return ("f32," if dtype == "f32" else "") + "paired:" + ":".join(str(int(x)) for d in descs for x in d)


def test_what_runs_together(checker):  # noqa: F811
    for form in ("dWhat", "dWhat +="):
        cases = [name(dt, desc(form, *s), desc("dXhat", *s)) for dt, *s in SHAPES]
        assert paired(checker, cases) == [int(x) for x in SHAPES.values()]
    assert paired(checker, [name("bf16", *aa_descs(*s)[1:]) for s in AA_SHAPES]) == [int(x) for x in AA_SHAPES.values()]
    # larger blocks, a product staged through registers beside one of the LDS-DMA kernels, the fp32 matrix instructions in bf16 stay apart
    apart = [("bf16", 2048, 513, 513, 32), ("bf16", 512, 192, 250, 32), ("bf16", 40, 6, 40, 8), ("f32", 512, 512, 512, 32)]
    assert paired(checker, [name(dt, desc("dWhat", *s), desc("dXhat", *s)) for dt, *s in apart]) == [0, 1, 0, 0]
    assert paired(checker, [name("bf16", desc("dWhat", 512, 192, 250, 32), desc("dXhat", 512, 192, 256, 32))]) == [0]


def test_contractions_that_groups_share(checker):  # noqa: F811
    """Of the products that run together, those that would be added up in another order by themselves."""
    def shared(descs):
        return any(path == "staged" and block.split(":")[1:] not in (["0"], ["1"]) for path, block in routes(checker, descs))
    layers = {s for s, together in SHAPES.items() if together and s[0] == "bf16" and shared([desc(f, *s[1:]) for f in ("dWhat", "dXhat")])}
    assert layers == SHARED
    assert {s for s, together in AA_SHAPES.items() if together and shared(aa_descs(*s)[1:])} == AA_SHARED


def test_edges_of_the_blocks(checker):  # noqa: F811
    """The shapes above reach all four pairs of block edges."""
    edges = set()
    for dt, *s in (s for s, together in SHAPES.items() if together and s[0] == "bf16" and s[2] % 8 == 0 and s[3] % 8 == 0):
        edges.add(tuple(b == "64x64" for _, b in routes(checker, [desc("dWhat", *s), desc("dXhat", *s)])))
    assert len(edges) == 4, edges


def test_pair_addresses(checker):  # noqa: F811
    checker(*(f"{'f32,' if dt == 'f32' else ''}bwd:{4 * M}:{4 * K}:{4 * N}:{r}" for dt, M, K, N, r in SHAPES),
            *(f"aa:{nb}:{4 * M}:{4 * K}:{4 * N}:{r}" for nb, M, K, N, r, _ in AA_SHAPES), "ragged:5:39:300:164:49", "f32,ragged:3:13:24:20:11",
            "ragged:9:50:44:1000:8")
