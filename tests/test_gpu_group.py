"""GPU parity of the group path: plans that compare most pairs of a set of dictionaries find the
shared k-mers of all pairs in one pass over the indexes.  Each case sits where that path changes
form -- items past its LDS arrays (taken in parts, or merged k-mer by k-mer), runs longer than a
descriptor's length field, multiplicities past a posting's bits, rows of more columns than a tile's
hash table, ties past the slab, tasks asking for one direction, 64-bit k-mer identities, empty and
tiny genomes, filters -- and must give the oracle's best hits and BBH, element by element."""
import random

import numpy as np
import pytest

import oracle
from helpers import check_bbh, check_bh
from synth import genome_from_strings, make_config

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU collection
    pytest.skip("needs the GPU", allow_module_level=True)

import paper_2510_23679_amd as pdp  # noqa: E402

AA = "ACDEFGHIKLMNPQRSTVWY"
BOTH = pdp.PDP_TASK_AB | pdp.PDP_TASK_BA | pdp.PDP_TASK_BBH


def _word(rng, n, letters=AA):
    return "".join(rng.choice(letters) for _ in range(n))


def _copies(rng, anc, sub, letters=AA):
    return ["".join(rng.choice(letters) if rng.random() < sub else c for c in s) for s in anc]


def _family(seed, genomes, genes, lo, hi, sub, letters=AA):
    rng = random.Random(seed)
    anc = [_word(rng, rng.randint(lo, hi), letters) for _ in range(genes)]
    out = []
    for _ in range(genomes):
        g = _copies(rng, anc, sub, letters) + [_word(rng, rng.randint(lo, hi), letters) for _ in range(genes // 5)]
        rng.shuffle(g)
        out.append(g)
    return out


def _shared_motif(seed, genomes, genes, motif, sub=0.1):
    # one motif in every gene of every genome: its k-mers have runs of genomes x genes postings
    rng = random.Random(seed)
    anc = [_word(rng, rng.randint(20, 60)) for _ in range(genes)]
    return [[s + motif for s in _copies(rng, anc, sub)] for _ in range(genomes)]


def _paralogs(seed):
    # six equal copies of every other gene: rows and columns with more ties than the slab keeps
    rng = random.Random(seed)
    anc = [_word(rng, rng.randint(30, 90)) for _ in range(40)]
    out = []
    for x in range(9):
        g = []
        for i, s in enumerate(_copies(rng, anc, 0.08)):
            g += [s] * (6 if i % 2 == x % 2 else 1)
        rng.shuffle(g)
        out.append(g)
    return out


def _counts(seed):
    # a letter repeated 40,000 times (multiplicities past a posting's bits), 300 and 20 times, and
    # pairs of genomes sharing a k-mer of which one side has 300
    rng = random.Random(seed)
    out = _family(seed, 16, 300, 20, 40, 0.1)
    for x in (0, 3, 4):
        out[x][7] = "A" * (40000 - x) + _word(rng, 30)
    out[1][9], out[2][9], out[6][11] = "A" * 300, "A" * 20 + _word(rng, 9), "C" * 300 + _word(rng, 9)
    out[7][3] = "C" * 6
    return out


def _uneven(seed):
    out = _family(seed, 14, 60, 20, 80, 0.1)
    out[2], out[5], out[9] = [], out[5][:1], ["ACD", ""] + out[9][:3]
    return out


CASES = {
    "family": (lambda: [[g for g in x.strings()] for x in make_config(2, genomes=9, genes=260).genomes], 5, "aa", {}),
    "family, 33 genomes": (lambda: _family(1, 33, 70, 20, 90, 0.12), 5, "aa", {}),
    "parts": (lambda: _family(2, 60, 260, 30, 60, 0.1), 6, "aa", {}),
    "merge and long runs": (lambda: _shared_motif(3, 9, 320, "WWWWWWWWW"), 5, "aa", {}),
    "long runs": (lambda: _shared_motif(4, 9, 40, "HHHKWWMMMCC"), 5, "aa", {}),
    "dense rows": (lambda: _shared_motif(5, 8, 2400, "MMMMMMMC", 0.3), 5, "aa", {}),
    "ties": (lambda: _paralogs(6), 5, "aa", {}),
    "ties, filters": (lambda: _paralogs(7), 5, "aa", {"theta": (3, 4), "tau": (1, 5)}),
    "dense rows, filters": (lambda: _shared_motif(8, 8, 2300, "MMMMMMMC", 0.3), 5, "aa",
                            {"theta": (1, 2), "tau": (1, 20)}),
    "counts": (lambda: _counts(9), 5, "aa", {}),
    "counts, filters": (lambda: _counts(9), 5, "aa", {"theta": (1, 2), "tau": (1, 5)}),
    "uneven": (lambda: _uneven(10), 4, "aa", {}),
    "35-bit codes": (lambda: _family(11, 9, 90, 30, 90, 0.08), 7, "aa", {}),
    "50-bit codes": (lambda: _family(12, 9, 90, 30, 90, 0.05), 10, "aa", {}),
    "60-bit codes": (lambda: _family(13, 9, 90, 40, 90, 0.04), 12, "aa", {}),
    "nucleotides": (lambda: _family(14, 9, 60, 60, 300, 0.08, "ACGT"), 10, "nt", {}),
    "nucleotides, 62-bit codes": (lambda: _family(15, 9, 60, 60, 300, 0.02, "ACGT"), 31, "nt", {}),
}


def _compare(og, pairs, res, flags, theta=None, tau=None):
    want = oracle.all_pairs_sparse(og, pairs, theta=theta, tau=tau)
    for t, (key, f) in enumerate(zip(pairs, flags)):
        ab, ba, bb = want[key]
        if f & pdp.PDP_TASK_AB:
            check_bh(res.best_hits(t, 0), ab)
        if f & pdp.PDP_TASK_BA:
            check_bh(res.best_hits(t, 1), ba)
        if f & pdp.PDP_TASK_BBH:
            check_bbh(res.bbh_pairs(t), bb)


def _grouped(plan, tasks):
    """Whether the plan takes another path than the persistent one, which joins pair by pair."""
    return plan.info.join_groups != pdp.Plan(tasks, pdp.params(persistent=True)).info.join_groups


@pytest.mark.parametrize("name", list(CASES))
def test_group_path(name):
    make, k, al, filters = CASES[name]
    genomes = [genome_from_strings(g, alphabet=al) for g in make()]
    print("[case]", name, "k", k, "genes", [g.n_genes for g in genomes], flush=True)
    dicts = [pdp.Dictionary.build_from(g, k) for g in genomes]
    pairs = [(i, j) for i in range(len(genomes)) for j in range(i + 1, len(genomes))]
    tasks = pdp.all_pairs_tasks(dicts, pairs)
    runner = pdp.PairRunner(tasks, pdp.params(**filters))
    assert _grouped(runner.plan, tasks)
    runner.ws.buf.fill_(255)
    og = oracle.genomes(genomes, k, alphabet=al)
    outs = []
    for _ in range(2):  # the second launch starts from what the first one left in the workspace
        runner.run()
        res = runner.results()
        outs.append(res)
    assert all(np.array_equal(x, y) for x, y in zip(outs[0].bh + outs[0].bbh, outs[1].bh + outs[1].bbh))
    _compare(og, pairs, outs[0], [BOTH] * len(pairs), filters.get("theta"), filters.get("tau"))


def test_group_path_one_direction_tasks_and_two_groups():
    # two groups of another k in one plan, the tasks of each asking for one direction, for both or
    # for BBH, named in both orders, and a pair that belongs to neither group
    parts = [(_family(21, 10, 50, 20, 70, 0.1), 5), (_family(22, 9, 70, 30, 60, 0.1), 6), (_family(23, 2, 40, 20, 50, 0.1), 5)]
    rng = random.Random(24)
    tasks, expect = [], []
    for genes, k in parts:
        genomes = [genome_from_strings(g) for g in genes]
        dicts = [pdp.Dictionary.build_from(g, k) for g in genomes]
        og = oracle.genomes(genomes, k)
        pairs = [(i, j) if rng.random() < 0.5 else (j, i) for i in range(len(genomes)) for j in range(i)]
        flags = [rng.choice([pdp.PDP_TASK_AB, pdp.PDP_TASK_BA, pdp.PDP_TASK_AB | pdp.PDP_TASK_BA, pdp.PDP_TASK_BBH])
                 for _ in pairs]
        tasks += [(dicts[i], dicts[j], f) for (i, j), f in zip(pairs, flags)]
        expect.append((og, pairs, [f | (3 if f & pdp.PDP_TASK_BBH else 0) for f in flags]))
    print("[case] one-direction tasks, two groups and a pair:", len(tasks), "tasks", flush=True)
    runner = pdp.PairRunner(tasks)
    assert _grouped(runner.plan, tasks)
    runner.run()
    res = runner.results()

    class Shifted:  # the results of a slice of the plan's tasks
        def __init__(self, first):
            self.first = first

        def best_hits(self, t, d):
            return res.best_hits(self.first + t, d)

        def bbh_pairs(self, t):
            return res.bbh_pairs(self.first + t)

    first = 0
    for og, pairs, flags in expect:
        _compare(og, pairs, Shifted(first), flags)
        first += len(pairs)


def test_group_path_grows_a_small_capacity():
    # the group path keeps no records; its column candidates share the record capacity
    genomes = [genome_from_strings(g) for g in _family(31, 9, 60, 20, 70, 0.1)]
    print("[case] group path, capacity 64", flush=True)
    dicts = [pdp.Dictionary.build_from(g, 5) for g in genomes]
    runner = pdp.PairRunner(pdp.all_pairs_tasks(dicts), pdp.params(inc_capacity=64))
    runner.launch()
    code, needed, where = pdp.read_status(runner.status)
    assert code == pdp.PDP_E_CAPACITY and where == 0 and needed > 64
    runner.run()
    pairs = [(i, j) for i in range(9) for j in range(i + 1, 9)]
    _compare(oracle.genomes(genomes, 5), pairs, runner.results(), [BOTH] * len(pairs))
