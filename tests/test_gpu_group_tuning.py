"""The autotuner on a collection whose tasks form a group: the launch shapes it would choose between are one
there, so one is timed, and the result does not name tile rows or sub-ranges that nothing used."""
import random

import pytest

from synth import genome_from_strings

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU collection
    pytest.skip("needs the GPU", allow_module_level=True)

import paper_2510_23679_amd as pdp  # noqa: E402


def _tasks():
    rng = random.Random(1)
    anc = ["".join(rng.choice("ACDEFGHIKLMNPQRSTVWY") for _ in range(60)) for _ in range(150)]
    genomes = [genome_from_strings(["".join(rng.choice("ACDEFGHIKLMNPQRSTVWY") if rng.random() < 0.1 else c for c in s)
                                    for s in anc]) for _ in range(24)]
    return pdp.all_pairs_tasks([pdp.Dictionary.build_from(g, 5) for g in genomes])


def test_group_candidates_are_timed_once():
    tasks = _tasks()
    group = [pdp.params(tile_rows=r, join_entries=j, colmax=c) for r in (64, 128) for j in (512, 768) for c in (False, True)]
    print("[case] autotuner, candidates on the group path", flush=True)
    best, res = pdp.autotune(tasks, group, reps=2)
    assert res.tried == 1
    assert (best.tile_rows, best.join_entries, best.lds_budget, best.flags) == (0, 0, 0, 0)
    best, res = pdp.autotune(tasks, group + [pdp.params(tile_rows=64, persistent=True)], reps=2)
    assert res.tried == 2
    runner = pdp.PairRunner(tasks, best)
    assert runner.run()[0] == 0
