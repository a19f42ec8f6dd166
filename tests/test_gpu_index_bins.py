"""GPU parity of the dictionary build where its index partition changes form: bins of 8-byte and of
16-byte records filled to their LDS and past it, slots of one thread's ranking and past it, small
and large placement blocks, and multiplicity vectors whose sorted keys pass through LDS in one part
or two.  Every array is compared with the oracle's."""
import random

import pytest

import oracle
from helpers import check_dictionary
from synth import genome_from_strings, random_genome

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU collection
    pytest.skip("needs the GPU", allow_module_level=True)

import paper_2510_23679_amd as pdp  # noqa: E402

AA = "ACDEFGHIKLMNPQRSTVWY"


def _skewed(seed, genes, motif, tail):
    # a motif at the head of every gene: its k-mers crowd one bucket, and one slot of its bin
    rng = random.Random(seed)
    return [motif + "".join(rng.choice(AA) for _ in range(rng.randint(*tail))) for _ in range(genes)]


def _lengths(k):
    # windows around the sort tiers of a wave (256, 512, 1024) and of a work-group (2048)
    rng = random.Random(7)
    return ["".join(rng.choice(AA) for _ in range(w + k - 1))
            for w in (1, 2, 63, 64, 65, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 2047, 2048, 2049)] + \
           ["A" * (w + k - 1) for w in (255, 512, 513, 1024, 1500)]


CASES = {
    "sort tiers, 32-bit keys": (lambda: _lengths(6), 6),
    "sort tiers, base-20 keys": (lambda: _lengths(7), 7),
    "sort tiers, 64-bit keys": (lambda: _lengths(9), 9),
    "slot of 32 and 33 entries": (lambda: _skewed(1, 32, "WWWWWW", (20, 60)) + _skewed(2, 33, "MMMMMM", (20, 60)), 6),
    "bin past the ranked slots": (lambda: _skewed(3, 3000, "WWWWWWW", (10, 30)), 7),
    "bin past LDS, 8-byte records": (lambda: _skewed(4, 6000, "WWWWWWWW", (8, 14)), 6),
    "bin past LDS, 16-byte records": (lambda: _skewed(5, 1500, "WWWWWWWWWW", (8, 14)), 9),
    "two-letter k-mers": (lambda: _skewed(6, 5000, "W", (4, 12)), 2),
}


@pytest.mark.parametrize("name", list(CASES))
def test_index_bins(name):
    make, k = CASES[name]
    genome = genome_from_strings(make())
    print("[case]", name, "genes", genome.n_genes, "k", k, flush=True)
    d = pdp.Dictionary.build_from(genome, k)
    d.check_status()
    check_dictionary(d.host(), oracle.OracleGenome(genome, k))


@pytest.mark.parametrize("k", [6, 7, 8])
def test_large_build_blocks(k):
    # past the size from which placement blocks are large, with a small genome among large ones
    genomes = [random_genome(40 + i, n, 200, 500) for i, n in enumerate((3500, 40, 4200))]
    print("[case] large build, k", k, [g.n_residues for g in genomes], flush=True)
    batch = pdp.DictionaryBatch([pdp.DeviceGenome.of(g) for g in genomes], k)
    batch.build()
    batch.check_status()
    for d, g in zip(batch.dicts, genomes):
        check_dictionary(d.host(), oracle.OracleGenome(g, k))
