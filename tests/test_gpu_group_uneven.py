"""The group path on letters used unevenly and on k-mers that many genes share: work items past their
LDS arrays (taken in ranges of buckets), buckets past them (in parts), hash slots from the size at which
their k-mers are merged one by one, runs that all waves of a tile walk, tiles past their hash table (in
the large one), items cut at letter boundaries.  Results against the oracle, or, where the oracle is too
slow, against the pair-by-pair join of the same dictionaries."""
import random
import statistics

import numpy as np
import pytest

import oracle
from helpers import check_bbh, check_bh
from synth import genome_from_strings

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU collection
    pytest.skip("needs the GPU", allow_module_level=True)

import paper_2510_23679_amd as pdp  # noqa: E402

AA = "ACDEFGHIKLMNPQRSTVWY"


def _word(rng, n, letters=AA):
    return "".join(rng.choice(letters) for _ in range(n))


def _family(seed, genomes, genes, lo, hi, letters=AA, sub=0.1, head="", heads=()):
    """Mutated copies of common ancestors; the first heads[x] genes of genome x begin with ``head``."""
    rng = random.Random(seed)
    anc = [_word(rng, rng.randint(lo, hi), letters) for _ in range(genes)]
    out = []
    for x in range(genomes):
        g = ["".join(rng.choice(letters) if rng.random() < sub else c for c in s) for s in anc]
        n = heads[x] if heads else 0
        g = [head + s if i < n else s for i, s in enumerate(g)]
        rng.shuffle(g)
        out.append(g)
    return out


def _share(total, genomes):
    return [total // genomes + (1 if x < total % genomes else 0) for x in range(genomes)]


def _prefix(seed, genomes, genes):
    # four leading letters common to all genes, different ones after them: a bucket of many k-mers
    rng = random.Random(seed)
    anc = ["WMCH" + _word(rng, 12) for _ in range(genes)]
    return [[s[:rng.choice((12, 14, 16))] for s in anc] for _ in range(genomes)]


MOTIF = "WMCHWM"
CASES = {
    # 8 of 20 letters: a bucket that is used holds 39 times the average
    "items in ranges of buckets": (lambda: _family(1, 9, 150, 40, 80, "ACDEFGHI", 0.3), 6, "aa", {}),
    "items in ranges of buckets, 64-bit identities": (lambda: _family(2, 9, 150, 40, 80, "ACDE", 0.3), 12, "aa", {}),
    "bucket in parts": (lambda: _prefix(3, 9, 320), 8, "aa", {}),
    "bucket in parts and a hot k-mer": (lambda: [g + [MOTIF + "CD"] * 60 for g in _prefix(4, 9, 260)], 6, "aa", {}),
    "slot of 511": (lambda: _family(5, 9, 90, 30, 60, head=MOTIF, heads=_share(511, 9)), 6, "aa", {}),
    "slot of 512": (lambda: _family(5, 9, 90, 30, 60, head=MOTIF, heads=_share(512, 9)), 6, "aa", {}),
    "slot of 512, 64-bit identities": (lambda: _family(6, 9, 90, 30, 60, head=MOTIF * 2, heads=_share(512, 9)), 12, "aa", {}),
    "run of 1023": (lambda: _family(7, 9, 130, 30, 60, head=MOTIF, heads=_share(1023, 9)), 6, "aa", {}),
    "run of 1024": (lambda: _family(7, 9, 130, 30, 60, head=MOTIF, heads=_share(1024, 9)), 6, "aa", {}),
    "tiles past the table": (lambda: _family(8, 9, 400, 30, 60, head=MOTIF, heads=[300] * 9), 6, "aa", {}),
    "tiles past the table, filters": (lambda: _family(8, 9, 400, 30, 60, head=MOTIF, heads=[300] * 9), 6, "aa",
                                      {"theta": (1, 2), "tau": (1, 20)}),
    "letter boundaries, k = 8": (lambda: _family(9, 9, 120, 40, 90, sub=0.05), 8, "aa", {}),
    "letter boundaries, k = 9": (lambda: _family(10, 9, 120, 40, 90, sub=0.05), 9, "aa", {}),
    "nucleotides, k = 24": (lambda: _family(11, 9, 60, 60, 300, "ACGT", 0.02), 24, "nt", {}),
    "nucleotides, k = 25": (lambda: _family(12, 9, 60, 60, 300, "ACGT", 0.02), 25, "nt", {}),
}


def _grouped(plan, tasks):
    return plan.info.join_groups != pdp.Plan(tasks, pdp.params(persistent=True)).info.join_groups


@pytest.mark.parametrize("name", list(CASES))
def test_against_the_oracle(name):
    make, k, al, filters = CASES[name]
    genomes = [genome_from_strings(g, alphabet=al) for g in make()]
    print("[case]", name, "k", k, "genes", [g.n_genes for g in genomes], flush=True)
    dicts = [pdp.Dictionary.build_from(g, k) for g in genomes]
    pairs = [(i, j) for i in range(len(genomes)) for j in range(i + 1, len(genomes))]
    tasks = pdp.all_pairs_tasks(dicts, pairs)
    runner = pdp.PairRunner(tasks, pdp.params(**filters))
    assert _grouped(runner.plan, tasks)
    runner.ws.buf.fill_(255)
    want = oracle.all_pairs_sparse(oracle.genomes(genomes, k, alphabet=al), pairs, **filters)
    for _ in range(2):  # the second launch starts from what the first one left in the workspace
        runner.run()
        res = runner.results()
        for t, key in enumerate(pairs):
            ab, ba, bb = want[key]
            check_bh(res.best_hits(t, 0), ab)
            check_bh(res.best_hits(t, 1), ba)
            check_bbh(res.bbh_pairs(t), bb)


def _same_as_pair_by_pair(genomes, k, **prm):
    dicts = [pdp.Dictionary.build_from(g, k) for g in genomes]
    tasks = pdp.all_pairs_tasks(dicts)
    got = pdp.PairRunner(tasks, pdp.params(**prm))
    assert _grouped(got.plan, tasks)
    got.run()
    want = pdp.PairRunner(tasks, pdp.params(persistent=True, **prm))
    want.run()
    for x, y in zip(got.results().bh + got.results().bbh, want.results().bh + want.results().bbh):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("genomes", [61, 128, 255])
def test_many_dictionaries(genomes):
    print("[case]", genomes, "dictionaries", flush=True)
    _same_as_pair_by_pair([genome_from_strings(g) for g in _family(21, genomes, 8, 20, 60, sub=0.15)], 5)


def test_rows_past_the_large_table():
    # 7 genomes of 7600 genes that all share one k-mer: with filters the large table holds 8192 sums
    rng = random.Random(22)
    genomes = []
    for _ in range(7):
        genes = [MOTIF + _word(rng, 3 if i else 1) for i in range(7600)]
        rng.shuffle(genes)
        genomes.append(genome_from_strings(genes))
    print("[case] rows past the large table", flush=True)
    _same_as_pair_by_pair(genomes, 6, theta=(1, 2))


def _device_us(launch):
    launch()
    times = []
    for _ in range(7):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        launch()
        b.record()
        torch.cuda.synchronize()
        times.append(1e3 * a.elapsed_time(b))
    return statistics.median(times)


def test_a_shared_motif_does_not_stall_the_launch():
    # a motif in 250 genes of each genome took 70 times the launch without it; pair by pair it takes 3
    rng = np.random.default_rng(23)
    letters = np.frombuffer(AA.encode(), np.uint8)
    times = []
    for motif in (0, 250):
        genomes = []
        for _ in range(10):
            genes = letters[rng.integers(0, 20, (3000, 300))]
            genes[:motif, 100:108] = np.frombuffer(b"WMCHWMCH", np.uint8)
            g = genome_from_strings(["A"])
            g.residues, g.offsets = genes.reshape(-1).copy(), np.arange(3001, dtype=np.uint64) * 300
            genomes.append(g)
        runner = pdp.PairRunner(pdp.all_pairs_tasks([pdp.Dictionary.build_from(g, 6) for g in genomes]))
        runner.run()
        times.append(_device_us(runner.launch))
    print("[case] launch", times, "us", flush=True)
    assert times[1] < 15 * times[0]
