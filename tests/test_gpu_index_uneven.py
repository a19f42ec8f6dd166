"""GPU parity of the dictionary build where the index partition is uneven: genomes of a few letters, or of
letters as often as in proteins, whose bins do not fit LDS (few parts, more parts than are laid out at a
time, single slots past LDS), and bins as many as the staged placement takes and more.  Every array is
compared with the oracle's."""
import statistics

import numpy as np
import pytest

import oracle
from helpers import check_dictionary
from synth import genome_from_strings

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU collection
    pytest.skip("needs the GPU", allow_module_level=True)

import paper_2510_23679_amd as pdp  # noqa: E402

AA = "ACDEFGHIKLMNPQRSTVWY"
# letters as often as in an average protein, in tenths of a percent
PROTEIN = [83, 14, 55, 67, 39, 71, 23, 59, 58, 97, 24, 41, 47, 39, 55, 67, 54, 69, 11, 29]


def _genome(seed, genes, length, letters, weights=None, alphabet="aa", head=""):
    rng = np.random.default_rng(seed)
    p = None if weights is None else np.asarray(weights) / np.sum(weights)
    x = np.frombuffer(letters.encode(), np.uint8)[rng.choice(len(letters), (genes, length), p=p)]
    if head:
        x[:, :len(head)] = np.frombuffer(head.encode(), np.uint8)
    g = genome_from_strings(["A"], alphabet=alphabet)
    g.residues, g.offsets = x.reshape(-1).copy(), np.arange(genes + 1, dtype=np.uint64) * np.uint64(length)
    return g


CASES = {
    "protein letters, 8-byte records": (lambda: _genome(1, 4300, 500, AA, PROTEIN), 6),
    "protein letters, base-20 keys": (lambda: _genome(2, 4300, 500, AA, PROTEIN), 7),
    "protein letters, 16-byte records": (lambda: _genome(3, 4300, 500, AA, PROTEIN), 8),
    "four letters: more parts than one layout": (lambda: _genome(4, 6000, 400, "ACDE"), 6),
    "four letters, 16-byte records": (lambda: _genome(5, 2000, 400, "ACDE"), 9),
    "slots past LDS": (lambda: _genome(6, 9000, 250, AA, PROTEIN, head="WWWWWWWWWW"), 6),
    "slots past LDS, 16-byte records": (lambda: _genome(7, 9000, 250, AA, PROTEIN, head="WWWWWWWWWWWW"), 9),
    "5000 bins, staged placement": (lambda: _genome(8, 13600, 500, AA), 6),
    "8192 bins, placement without staging": (lambda: _genome(9, 11200, 1000, "ACGT", alphabet="nt"), 13),
}


@pytest.mark.parametrize("name", list(CASES))
def test_uneven_bins(name):
    make, k = CASES[name]
    genome = make()
    print("[case]", name, "genes", genome.n_genes, "letters", genome.n_residues, "k", k, flush=True)
    d = pdp.Dictionary.build_from(genome, k)
    d.check_status()
    check_dictionary(d.host(), oracle.OracleGenome(genome, k))


def _build_us(weights):
    batch = pdp.DictionaryBatch([pdp.DeviceGenome.of(_genome(20 + i, 4900, 340, AA, weights)) for i in range(10)], 6)
    batch.build()
    times = []
    for _ in range(7):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        batch.build()
        b.record()
        torch.cuda.synchronize()
        times.append(1e3 * a.elapsed_time(b))
    return statistics.median(times)


def test_protein_letters_do_not_slow_the_build_down():
    # the bins past LDS, sorted in global memory, made this build four times as long as that of even letters
    even, protein = _build_us(None), _build_us(PROTEIN)
    print("[case] build", even, protein, "us", flush=True)
    assert protein < 2 * even


@pytest.mark.parametrize("k", [6, 7, 8])
@pytest.mark.parametrize("letters", [655359, 655360])
def test_around_the_small_builds(letters, k):
    # a build's letters and one entry per genome: up to 40 blocks of 16384 take the small forms
    genome = _genome(30, 1, letters % 1000 or 1000, AA, PROTEIN)
    rest = _genome(31, letters // 1000, 1000, AA, PROTEIN)
    genome.residues = np.concatenate([rest.residues, genome.residues])[:letters]
    genome.offsets = np.append(rest.offsets, np.uint64(letters)) if letters % 1000 else rest.offsets
    print("[case] small builds,", letters, "letters, k", k, flush=True)
    d = pdp.Dictionary.build_from(genome, k)
    d.check_status()
    check_dictionary(d.host(), oracle.OracleGenome(genome, k))


@pytest.mark.parametrize("k,letters", [(k, n) for k in (6, 7) for n in (20, 60, 130, 250, 500)])
def test_sub_slots_of_part_of_a_letter(k, letters):
    # genomes of 20,000 to 500,000 letters beside one that makes the build large: bins of 16384 to 512 buckets,
    # whose slots take none to four bits of the next letter
    genomes = [_genome(32 + i, letters, 1000 + i, AA, PROTEIN) for i in range(3)] + [_genome(40, 1000, 700, AA)]
    print("[case] sub-slots, k", k, [g.n_residues for g in genomes], flush=True)
    batch = pdp.DictionaryBatch([pdp.DeviceGenome.of(g) for g in genomes], k)
    batch.build()
    batch.check_status()
    for d, g in zip(batch.dicts, genomes):
        check_dictionary(d.host(), oracle.OracleGenome(g, k))


@pytest.mark.parametrize("k", [11, 13, 17])
def test_sub_slots_of_part_of_a_letter_nucleotides(k):
    genomes = [_genome(60 + n, n, 1001, "ACGT", alphabet="nt") for n in (50, 200, 400, 900)]
    print("[case] nucleotide sub-slots, k", k, [g.n_residues for g in genomes], flush=True)
    batch = pdp.DictionaryBatch([pdp.DeviceGenome.of(g) for g in genomes], k)
    batch.build()
    batch.check_status()
    for d, g in zip(batch.dicts, genomes):
        check_dictionary(d.host(), oracle.OracleGenome(g, k))


def test_a_genome_of_ordinary_size_takes_the_large_forms():
    # with small blocks and bins 1.46 million letters took 2.5 times as long as 0.34 million, with large ones 1.4
    def build(genes):
        batch = pdp.DictionaryBatch([pdp.DeviceGenome.of(_genome(50, genes, 340, AA))], 6)
        batch.build()
        times = []
        for _ in range(9):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            batch.build()
            b.record()
            torch.cuda.synchronize()
            times.append(1e3 * a.elapsed_time(b))
        return statistics.median(times)

    few, many = build(1000), build(4300)
    print("[case] build", few, many, "us", flush=True)
    assert many < 1.9 * few
