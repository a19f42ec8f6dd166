"""The record capacity of plans that take the group path.  Candidates for column maxima are listed as tiles
reach them, so their number depends on the order of the tiles; whether a plan fits its capacity must not:
past the list the tiles are replayed against the final maxima, and the hits, whose number the oracle knows,
are what has to fit.  What the pair-by-pair join accepts is accepted."""
import random

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
SLAB = 4  # hits a row keeps outside the candidates


def _word(rng, n):
    return "".join(rng.choice(AA) for _ in range(n))


def _paralogs(seed, genomes=9, families=40, copies=6, length=(30, 90), motif=""):
    # copies of half the genes: rows and columns with more ties than the slab keeps
    rng = random.Random(seed)
    anc = [_word(rng, rng.randint(*length)) + motif for _ in range(families)]
    out = []
    for x in range(genomes):
        g = []
        for i, s in enumerate(anc):
            m = "".join(rng.choice(AA) if rng.random() < 0.08 else c for c in s)
            g += [m] * (copies if i % 2 == x % 2 else 1)
        rng.shuffle(g)
        out.append(g)
    return [genome_from_strings(g) for g in out]


def _hits(want, pairs):
    """Hits that leave through the column maxima: the second genome's, and rows of more ties than SLAB."""
    n = 0
    for p in pairs:
        ab, ba, _ = want[p]
        rows = ab.ptr[1:] - ab.ptr[:-1]
        n += int(ba.ptr[-1]) + int(rows[rows > SLAB].sum())
    return n


def _setup(genomes, k, **filters):
    dicts = [pdp.Dictionary.build_from(g, k) for g in genomes]
    pairs = [(i, j) for i in range(len(genomes)) for j in range(i + 1, len(genomes))]
    return dicts, pairs, oracle.all_pairs_sparse(oracle.genomes(genomes, k), pairs, **filters)


def _check(runner, pairs, want):
    res = runner.results()
    for t, p in enumerate(pairs):
        ab, ba, bb = want[p]
        check_bh(res.best_hits(t, 0), ab)
        check_bh(res.best_hits(t, 1), ba)
        check_bbh(res.bbh_pairs(t), bb)


CASES = {
    "ties": (lambda: _paralogs(1), 5, {}),
    "ties, filters": (lambda: _paralogs(2), 5, {"theta": (3, 4), "tau": (1, 5)}),
    "rows past the table": (lambda: _paralogs(3, 8, 1400, 2, (12, 20), "MMMMMMMC"), 5, {}),
    "rows past the table, filters": (lambda: _paralogs(4, 8, 1400, 2, (12, 20), "MMMMMMMC"), 5, {"theta": (1, 2)}),
}


@pytest.mark.parametrize("name", list(CASES))
def test_a_plan_fits_exactly_its_hits(name):
    make, k, filters = CASES[name]
    genomes = make()
    print("[case]", name, [g.n_genes for g in genomes], flush=True)
    dicts, pairs, want = _setup(genomes, k, **filters)
    hits = _hits(want, pairs)
    tasks = pdp.all_pairs_tasks(dicts, pairs)
    assert pdp.Plan(tasks).info.tiles != pdp.Plan(tasks, pdp.params(persistent=True)).info.tiles  # the group path
    for cap, colmax in ((hits, False), (hits - 1, False), ((hits + 1) // 2, True), ((hits - 1) // 2, True)):
        runner = pdp.PairRunner(tasks, pdp.params(inc_capacity=cap, colmax=colmax, **filters),
                                *[8 * sum(g.n_genes for g in genomes) * len(genomes)] * 2)
        fits = cap * (2 if colmax else 1) >= hits
        for _ in range(3):
            runner.launch()
            code, needed, where = pdp.read_status(runner.status)
            assert (code, needed, where) == ((0, 0, 2**64 - 1) if fits else (pdp.PDP_E_CAPACITY, hits, 0)), (cap, colmax)
        if fits:
            _check(runner, pairs, want)
        runner.run()  # grows where it has to
        _check(runner, pairs, want)


def test_a_group_beside_pairs_with_column_maxima():
    # the pairs' candidates and the group's have their own places and counts
    genomes, others = _paralogs(5), _paralogs(6, 2)
    dicts, pairs, want = _setup(genomes, 5)
    odicts, opairs, owant = _setup(others, 6)
    print("[case] a group beside a pair", flush=True)
    tasks = pdp.all_pairs_tasks(dicts, pairs) + pdp.all_pairs_tasks(odicts, opairs)
    runner = pdp.PairRunner(tasks, pdp.params(colmax=True, inc_capacity=max(_hits(want, pairs), 20000)))
    small = pdp.PairRunner(tasks, pdp.params(colmax=True, inc_capacity=64))
    for r in (runner, small):
        for _ in range(2):
            r.run()
            _check(r, pairs, want)
            res = r.results()
            ab, ba, bb = owant[(0, 1)]
            check_bh(res.best_hits(len(pairs), 0), ab)
            check_bh(res.best_hits(len(pairs), 1), ba)
            check_bbh(res.bbh_pairs(len(pairs)), bb)


def test_what_fits_by_pairs_fits():
    # the pair-by-pair join's own count of records, with and without column maxima
    genomes = _paralogs(7)
    dicts, pairs, want = _setup(genomes, 5)
    tasks = pdp.all_pairs_tasks(dicts, pairs)
    print("[case] what fits by pairs", flush=True)
    for colmax in (False, True):
        by_pairs = pdp.PairRunner(tasks, pdp.params(inc_capacity=1, persistent=True, colmax=colmax))
        by_pairs.launch()
        code, records, where = pdp.read_status(by_pairs.status)
        assert code == pdp.PDP_E_CAPACITY and where == 0
        runner = pdp.PairRunner(tasks, pdp.params(inc_capacity=records, colmax=colmax),
                                *[8 * sum(g.n_genes for g in genomes) * len(genomes)] * 2)
        for _ in range(3):
            runner.launch()
            assert pdp.read_status(runner.status)[0] == 0
        _check(runner, pairs, want)
