"""Last rounds of the 256 x 256 blocks: which are dealt out in parts, and their addresses (see test_cpu_address_check.py)."""
from test_cpu_address_check import checker, pytestmark  # noqa: F401
from test_cpu_routes import FORMS, desc, routes

from test_gpu_split import FEW, SHAPES


def split(run, descs):
    _, text = run(*("split:" + ":".join(map(str, d)) for d in descs))
    return [ln.split()[1] for ln in text.splitlines() if ln.startswith("  route")]


def test_parts_of_the_last_round(checker):  # noqa: F811
    for s, want in SHAPES.items():
        descs = [desc(f, *s) for f in FORMS]
        assert tuple(split(checker, descs)) == want, s
        for parts, (path, block) in zip(want, routes(checker, descs)):
            assert parts == "whole" or (path in ("wide", "pipe") and block == "256x256"), s
        # the same planes a few at a time are not cut, and stay with the kernels that add up in that order
        few = [desc(f, *s[:3], n) for f, parts in zip(FORMS, want) if parts != "whole" for n in {FEW, s[3] % FEW or FEW}]
        assert set(split(checker, few)) == {"whole"} and {path for path, _ in routes(checker, few)} <= {"wide", "pipe"}, s
    # whole rounds, less than one, a last one that is nearly full, contractions without whole lines, stacked problems: as they are
    stacked = list(desc("Yhat", 640, 64, 264, 64))
    stacked[-1] = 2
    assert split(checker, [desc("Yhat", 2048, 1024, 1024, 32), desc("Yhat", 256, 1024, 1024, 32), desc("dXhat", 1024, 1024, 1024, 31),
                           desc("Yhat", 648, 72, 264, 64), tuple(stacked)]) == ["whole"] * 5


def test_part_addresses(checker):  # noqa: F811
    checker(*(f"bwd:{4 * M}:{4 * K}:{4 * N}:{r}" for M, K, N, r in SHAPES))
