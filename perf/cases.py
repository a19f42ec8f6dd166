"""The work that users of this package have it do, as cases that can be timed.

A case is one call path through the public Python entry points: building k-mer dictionaries,
one pair of genomes, all pairs of a collection, many independent collections in one launch,
candidate filters and families, the long-gene path, and serving arriving genomes.  Genomes are
drawn on the GPU from a family model: a family's members are copies of one random ancestor with
substitutions and single-letter indels, gene lengths follow a lognormal law (median 300 amino
acids or 900 nucleotides, sigma 0.5, clipped), gene order is shuffled, and part of the genes are
exact copies of others (paralogs), half of them then carrying one substitution.

``listed`` names the cases, ``draw`` gives more of the same ranges, ``prepare`` makes the state
that a program holds before the call, ``run`` makes one call, ``work`` counts the bytes the call
cannot do without, and ``exact`` computes the same outputs with plain torch operations.
"""
import math
import random

import numpy as np
import torch

import paper_2510_23679_amd as pdp

LETTERS = {"aa": "ACDEFGHIKLMNPQRSTVWY", "nt": "ACGT"}
BITS = {"aa": 5, "nt": 2}
LEAD = {"aa": 4, "nt": 9}
# gene lengths: median, shortest, longest
LENGTHS = {"aa": (300.0, 50, 2000), "nt": (900.0, 150, 6000)}
SIGMA = 0.5


def listed():
    return [
        # An arriving genome's dictionary: the smallest genome sizes, one build at a time.
        {"name": "build_one_aa", "kind": "build", "genomes": 1, "genes": 1503, "spread": 0, "alphabet": "aa", "k": 7},
        # Dictionaries of a handful of genomes in one call, with the k of a larger collection
        # whose codes pass 35 bits.
        {"name": "build_six_aa_k8", "kind": "build", "genomes": 6, "genes": 3100, "spread": 2600, "alphabet": "aa",
         "k": 8},
        # One nucleotide genome, coding sequences of a bacterium of 4000 genes.
        {"name": "build_one_nt", "kind": "build", "genomes": 1, "genes": 4000, "spread": 0, "alphabet": "nt", "k": 13},
        # Two small genomes whose dictionaries stay: every launch of a plan, latency counts.
        {"name": "pair_200", "kind": "pairs", "genomes": 2, "genes": 200, "spread": 0, "alphabet": "aa", "k": 4,
         "core": 0.75, "paralogs": 0.0, "build": False, "colmax": False, "tile_rows": 0, "filters": False,
         "families": False},
        # The convenience calls, each with its own plan and checks: best hits both ways, then BBH.
        {"name": "calls_2x1001", "kind": "calls", "genomes": 2, "genes": 1001, "spread": 0, "alphabet": "aa", "k": 5},
        # A small collection, dictionaries and all pairs each step, the library's default parameters.
        {"name": "all_10x3000", "kind": "pairs", "genomes": 10, "genes": 3000, "spread": 0, "alphabet": "aa", "k": 6,
         "core": 0.6, "paralogs": 0.0, "build": True, "colmax": False, "tile_rows": 0, "filters": False,
         "families": False},
        # The same collection as nucleotides.
        {"name": "all_10x3000_nt", "kind": "pairs", "genomes": 10, "genes": 3000, "spread": 0, "alphabet": "nt",
         "k": 13, "core": 0.6, "paralogs": 0.0, "build": True, "colmax": False, "tile_rows": 0, "filters": False,
         "families": False},
        # The benchmark's collection: 50 genomes of 3000 to 5000 genes with paralogs, column maxima.
        {"name": "all_50x4000", "kind": "pairs", "genomes": 50, "genes": 4000, "spread": 1000, "alphabet": "aa",
         "k": 7, "core": 0.45, "paralogs": 0.05, "build": True, "colmax": True, "tile_rows": 128, "filters": False,
         "families": False},
        # Length and directional filters, families of the result, genomes of uneven sizes.
        {"name": "filtered_9x2477", "kind": "pairs", "genomes": 9, "genes": 2477, "spread": 1900, "alphabet": "aa",
         "k": 6, "core": 0.3, "paralogs": 0.05, "build": False, "colmax": False, "tile_rows": 0, "filters": True,
         "families": True},
        # Independent collections, each with its own k, built and compared in one launch.
        {"name": "batch_of_7", "kind": "batch", "instances": 7, "genomes": 17, "genes": 2750, "spread": 2250,
         "alphabet": "aa", "core": 0.5, "paralogs": 0.0},
        # A genome pair with genes past 65,535 windows.
        {"name": "long_genes_2x700", "kind": "long", "genomes": 2, "genes": 700, "spread": 0, "alphabet": "aa", "k": 6,
         "longest": 70001},
        # Genomes arriving at a server of resident genomes, four at a time, results fetched.
        {"name": "serve_4_of_60", "kind": "serve", "genomes": 60, "genes": 3000, "spread": 0, "alphabet": "aa", "k": 7,
         "arrivals": 4, "arrive_lo": 1000, "arrive_hi": 6000},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["build", "pairs", "pairs", "pairs", "pairs", "calls", "batch", "long", "serve"])
    al = rng.choice(["aa", "aa", "aa", "nt"]) if kind in ("build", "pairs", "calls") else "aa"
    if kind == "build":
        n, genes = _log_int(rng, 1, 6), _log_int(rng, 200, 5790)
        k = rng.randint(4, 9) if al == "aa" else rng.randint(10, 17)
        return {"kind": kind, "genomes": n, "genes": genes, "spread": genes // 4 if n > 1 else 0, "alphabet": al, "k": k}
    if kind == "calls":
        genes = _log_int(rng, 150, 5000)
        return {"kind": kind, "genomes": 2, "genes": genes, "spread": genes // 5, "alphabet": al,
                "k": _k_rule(2 * genes, al)}
    if kind == "batch":
        return {"kind": kind, "instances": rng.randint(2, 7), "genomes": rng.randint(4, 17),
                "genes": rng.randint(1500, 2750), "spread": rng.randint(0, 1000), "alphabet": al,
                "core": round(rng.uniform(0.3, 0.6), 2), "paralogs": 0.0}
    if kind == "long":
        return {"kind": kind, "genomes": 2, "genes": _log_int(rng, 50, 700), "spread": 0, "alphabet": al,
                "k": rng.randint(5, 7), "longest": rng.randint(66000, 70001)}
    if kind == "serve":
        lo = _log_int(rng, 300, 2000)
        return {"kind": kind, "genomes": rng.randint(8, 60), "genes": rng.randint(1000, 3000), "spread": 0,
                "alphabet": al, "k": 7, "arrivals": rng.randint(1, 4), "arrive_lo": lo, "arrive_hi": 2 * lo}
    genes, more = _log_int(rng, 200, 4000), rng.choice([0, 0, 0, 1])
    n = max(2, min(_log_int(rng, 2, 50 if al == "aa" else 10), (60000 if more else 130000) // genes))
    return {"kind": kind, "genomes": n, "genes": genes, "spread": int(genes * rng.uniform(0, 0.5)), "alphabet": al,
            "k": _k_rule(n * genes, al) + more, "core": round(rng.uniform(0.2, 0.5), 2),
            "paralogs": rng.choice([0.0, 0.05]), "build": rng.random() < 0.7, "colmax": rng.random() < 0.5,
            "tile_rows": rng.choice([0, 0, 64, 128]), "filters": rng.random() < 0.15, "families": rng.random() < 0.15}


def _k_rule(genes, alphabet):
    median = LENGTHS[alphabet][0]
    return pdp.k_rule(int(genes * median * 1.13), len(LETTERS[alphabet]))


# ------------------------------------------------------------------ genomes

class _Genome:
    """Letters and gene offsets on the host, as DeviceGenome and Server take them."""

    def __init__(self, residues, offsets, alphabet):
        self.residues = residues.cpu().numpy()
        self.offsets = offsets.cpu().numpy().astype("uint64")
        self.alphabet = alphabet


class _Model:
    """A family model: ancestors drawn once, genomes drawn from them."""

    def __init__(self, gen, alphabet, families, longest=0):
        self.gen, self.alphabet, self.dev = gen, alphabet, gen.device
        self.sigma, self.longest = len(LETTERS[alphabet]), longest
        self.ascii = torch.tensor(list(LETTERS[alphabet].encode()), dtype=torch.uint8, device=self.dev)
        lens = self._lengths(families)
        if longest:
            lens[:2] = torch.tensor([longest, longest - 997], device=self.dev)[: lens.numel()]
        self.off = _offsets(lens)  # the two longest genes, if any, are in every genome's core
        self.sym = self._letters(int(self.off[-1]))

    def _rand(self, n):
        return torch.rand(n, generator=self.gen, device=self.dev)

    def _letters(self, n):
        return torch.randint(0, self.sigma, (n,), generator=self.gen, device=self.dev, dtype=torch.int32)

    def _lengths(self, n):
        median, lo, hi = LENGTHS[self.alphabet]
        z = torch.randn(n, generator=self.gen, device=self.dev)
        return (median * torch.exp(SIGMA * z)).round().clamp(lo, hi).long()

    def members(self, which, sub_lo=0.05, sub_hi=0.30, indel_hi=0.03):
        """Members of families ``which``: each with its own substitution and indel rate."""
        n = which.numel()
        src, off = _gather(self.sym, self.off, which)
        gene = _gene_of(off)
        total = src.numel()
        sub = (sub_lo + (sub_hi - sub_lo) * self._rand(n))[gene]
        indel = (indel_hi * self._rand(n))[gene]
        hit = self._rand(total) < sub
        shift = 1 + torch.randint(0, self.sigma - 1, (total,), generator=self.gen, device=self.dev, dtype=torch.int32)
        sym = torch.where(hit, (src + shift) % self.sigma, src)
        event, side = self._rand(total) < indel, self._rand(total) < 0.5
        copies = 1 + (event & side).long() - (event & ~side).long()
        out = sym.repeat_interleave(copies)
        end = copies.cumsum(0)
        slots = end[event & side] - 1
        out[slots] = self._letters(slots.numel())
        cum = torch.cat([end.new_zeros(1), end])
        return out, cum[off]

    def letters_of(self, n_genes):
        median, lo, hi = LENGTHS[self.alphabet]
        return int(n_genes * median * 1.13) + 2 * self.longest

    def genome(self, n_genes, core, paralogs):
        """A genome: the core families, others drawn from the rest, singletons, copies."""
        families = self.off.numel() - 1
        dup = int(round(paralogs * n_genes))
        n_core = min(core, n_genes - dup)
        rest = n_genes - dup - n_core
        n_acc = min(int(0.75 * rest), families - n_core)
        acc = n_core + torch.randperm(families - n_core, generator=self.gen, device=self.dev)[:n_acc]
        sym, off = self.members(torch.cat([torch.arange(n_core, device=self.dev), acc]))
        lens = self._lengths(rest - n_acc)
        sym = torch.cat([sym, self._letters(int(lens.sum()))])
        off = torch.cat([off, off[-1] + _offsets(lens)[1:]])
        if dup:
            which = torch.randperm(off.numel() - 1, generator=self.gen, device=self.dev)[:dup]
            dsym, doff = _gather(sym, off, which)
            near = doff[: dup // 2] + (self._rand(dup // 2) * (doff[1 : dup // 2 + 1] - doff[: dup // 2])).long()
            dsym[near] = (dsym[near] + 1) % self.sigma
            sym, off = torch.cat([sym, dsym]), torch.cat([off, off[-1] + doff[1:]])
        return self.shuffled(sym, off)

    def shuffled(self, sym, off):
        """The genes in random order, their ends trimmed or extended by a few letters each so that
        genomes of the same number of genes hold the same number of letters."""
        n = off.numel() - 1
        order = torch.randperm(n, generator=self.gen, device=self.dev)
        sym, off = _gather(sym, off, order)
        lens = off.diff()
        more = self.letters_of(n) - int(lens.sum())
        each = more // n + (torch.arange(n, device=self.dev) < more % n).long()
        new = _offsets(lens + each)
        gene = _gene_of(new)
        inside = torch.arange(int(new[-1]), device=self.dev) - new[gene]
        old = (off[gene] + inside).clamp(max=sym.numel() - 1)
        sym, off = torch.where(inside < lens[gene], sym[old], self._letters(gene.numel())), new
        return _Genome(self.ascii[sym.long()], off, self.alphabet)


def _offsets(lens):
    return torch.cat([lens.new_zeros(1), lens.cumsum(0)])


def _gene_of(off):
    return torch.arange(off.numel() - 1, device=off.device).repeat_interleave(off.diff())


def _gather(sym, off, which):
    lens = off.diff()[which]
    new = _offsets(lens)
    at = torch.arange(int(new[-1]), device=sym.device) + (off[which] - new[:-1]).repeat_interleave(lens)
    return sym[at], new


def _generator(seed, stream=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1000003 + 7919 * stream + 17)
    return g


def _sizes(n, genes, spread):
    """Genes per genome, evenly over genes +- spread in a mixed order."""
    at = random.Random(n * 7919 + genes).sample(range(n), n)
    return [max(2, int(round(genes - spread + 2 * spread * (i + 0.5) / n))) for i in at]


def _collection(case, seed, stream=0, core_share=None):
    gen = _generator(seed, stream)
    sizes = _sizes(case["genomes"], case["genes"], case["spread"])
    core = int(min(sizes) * (case.get("core", 0.6) if core_share is None else core_share))
    families = core + max(sizes) + sum(sizes) // 20
    model = _Model(gen, case["alphabet"], families, case.get("longest", 0))
    return model, [model.genome(s, core, case.get("paralogs", 0.0)) for s in sizes], core


# -------------------------------------------------------------------- cases

def prepare(case, seed):
    return {"build": _prepare_build, "pairs": _prepare_pairs, "calls": _prepare_calls, "batch": _prepare_batch,
            "long": _prepare_pairs, "serve": _prepare_serve}[case["kind"]](case, seed)


def _prepare_build(case, seed):
    _, genomes, _ = _collection(case, seed)
    batch = pdp.DictionaryBatch([pdp.DeviceGenome.of(g) for g in genomes], case["k"])
    for d in batch.dicts:
        d.arena.zero_()
    return {"case": case, "batch": batch}


def _params(case):
    k = case["k"]
    filters = {"theta": (1, 2), "tau": (1, k)} if case.get("filters") else {}
    return pdp.params(tile_rows=case.get("tile_rows", 0), colmax=case.get("colmax", False), **filters)


def _cleared(runner):
    """Every entry of the outputs written, so that the part past the used entries compares equal."""
    for t in (runner.bh.col, runner.bh.num, runner.bh.den, runner.bbh.a, runner.bbh.b, runner.bbh.num, runner.bbh.den):
        t.zero_()
    return runner


def _prepare_pairs(case, seed):
    _, genomes, _ = _collection(case, seed)
    batch = pdp.DictionaryBatch([pdp.DeviceGenome.of(g) for g in genomes], case["k"])
    batch.build()
    runner = pdp.PairRunner(pdp.all_pairs_tasks(batch.dicts), _params(case))
    if not _checked(case):
        runner.run()  # sizes the buffers; the steps then launch without looking
    _cleared(runner)
    bases = [0]
    for d in batch.dicts:
        bases.append(bases[-1] + d.n_genes)
    return {"case": case, "batch": batch, "runner": runner, "bases": bases}


def _checked(case):
    """Whether a call goes through the runner's checked form, which waits for the status: a
    program that compares a collection once does, one that steps or keeps its plan does not."""
    return not case.get("build", False) and case["genes"] > 400


def _prepare_calls(case, seed):
    _, genomes, _ = _collection(case, seed)
    dicts = [pdp.Dictionary.build_from(g, case["k"]) for g in genomes]
    return {"case": case, "dicts": dicts}


def _batch_ks(case):
    return [_k_rule(case["genomes"] * case["genes"], case["alphabet"]) + i % 2 for i in range(case["instances"])]


def _batch_genomes(case, seed):
    out = []
    for i in range(case["instances"]):
        _, genomes, _ = _collection(dict(case, genomes=max(4, case["genomes"] - i)), seed, stream=i + 1)
        out.append(genomes)
    return out


def _prepare_batch(case, seed):
    every, ks, starts = [], [], [0]
    for genomes, k in zip(_batch_genomes(case, seed), _batch_ks(case)):
        every += [pdp.DeviceGenome.of(g) for g in genomes]
        ks += [k] * len(genomes)
        starts.append(len(every))
    batch = pdp.DictionaryBatch(every, ks)
    tasks = [t for lo, hi in zip(starts, starts[1:]) for t in pdp.all_pairs_tasks(batch.dicts[lo:hi])]
    batch.build()
    runner = pdp.PairRunner(tasks, pdp.params(colmax=True))
    runner.run()
    return {"case": case, "batch": batch, "runner": _cleared(runner)}


def _prepare_serve(case, seed):
    model, genomes, core = _collection(case, seed)
    families = model.off.numel() - 1
    arrivals = []
    for n in _sizes(case["arrivals"], (case["arrive_lo"] + case["arrive_hi"]) // 2,
                    (case["arrive_hi"] - case["arrive_lo"]) // 2):
        which = torch.randint(0, families, (n,), generator=model.gen, device=model.dev)
        arrivals.append(model.shuffled(*model.members(which)))
    batch = pdp.DictionaryBatch([pdp.DeviceGenome.of(g) for g in genomes], case["k"])
    batch.build()
    server = pdp.Server(batch.dicts, 6 << 30, slots=2, prm=pdp.params(colmax=True, tile_rows=128))
    return {"case": case, "batch": batch, "server": server, "arrivals": arrivals, "next": 0}


def _arrays(d):
    """The arrays of a built dictionary, views of its arena as pdp.h lays them out."""
    out = []
    for ptr, count, dtype in ((d.d.nwin, d.n_genes, torch.int32), (d.d.mv_ptr, d.n_genes + 1, torch.int32),
                              (d.d.mv_code, d.d.capacity, torch.int64), (d.d.mv_cnt, d.d.capacity, torch.int32),
                              (d.d.ix_dir, d.d.n_buckets + 1, torch.int32), (d.d.ix_code, d.d.capacity, torch.int64),
                              (d.d.ix_gene, d.d.capacity, torch.int32), (d.d.ix_cnt, d.d.capacity, torch.int32),
                              (d.d.ix_key, d.d.capacity, torch.int32)):
        at = ptr - d.arena.data_ptr()
        out.append(d.arena[at : at + count * dtype.itemsize].view(dtype))
    return out


def run(state):
    kind = state["case"]["kind"]
    if kind == "build":
        state["batch"].build()
        return [_arrays(d) for d in state["batch"].dicts]
    if kind == "calls":
        a, b = state["dicts"]
        ab, ba = pdp.bh(a, b), pdp.bh(b, a)
        both = pdp.bbh(ab, ba)
        return [_fixed(x.host(), x.n_rows) for x in (ab, ba, both)]
    if kind == "serve":
        return _serve(state)
    runner = state["runner"]
    if state["case"].get("build", kind == "batch"):
        state["batch"].build()
    if kind == "batch" or not _checked(state["case"]):
        runner.launch()
    else:
        runner.run()
    out = [[runner.bh.ptr, runner.bh.col, runner.bh.num, runner.bh.den],
           [runner.bbh.ptr, runner.bbh.a, runner.bbh.b, runner.bbh.num, runner.bbh.den]]
    if state["case"].get("families"):
        out.append(runner.families([state["bases"][i] for i, _ in _pairs(state["case"]["genomes"])],
                                   [state["bases"][j] for _, j in _pairs(state["case"]["genomes"])],
                                   state["bases"][-1]))
    return out


def _fixed(arrays, rows):
    """Host arrays of a CSR, its entries in two parts of fixed sizes, the second filled up with zeros."""
    head, out = rows * 3 // 4, [arrays[0]]
    for a in arrays[1:]:
        if a.size < head:
            a = np.concatenate([a, np.zeros(head - a.size, a.dtype)])
        tail = np.zeros(2 * rows + 1024 - head, a.dtype)
        tail[: a.size - head] = a[head:]
        out += [a[:head], tail]
    return out


def _pairs(n):
    return [(i, j) for i in range(n) for j in range(i + 1, n)]


def _serve(state):
    server, first = state["server"], state["next"]
    for i, g in enumerate(state["arrivals"]):
        server.submit(g, first + i)
    state["next"] = first + len(state["arrivals"])
    left = len(state["arrivals"])
    while left:
        left -= len(server.poll(max_n=8, wait_us=20000))
    out = []
    for i in range(len(state["arrivals"])):
        r = server.fetch(first + i)
        server.release(first + i)
        if r.code:
            raise RuntimeError(f"request {i}: code {r.code}")
        out.append([_fixed(r.bh, r.bh[0].size - 1), _fixed(r.bbh, r.bbh[0].size - 1)])
    return out


def work(case):
    """Bytes one call cannot do without: residues read, dictionaries written and read once, best
    hits and BBH pairs written (16 bytes each, about one per gene and direction)."""
    mean = LENGTHS[case["alphabet"]][0] * math.exp(SIGMA * SIGMA / 2)
    genes = case["genomes"] * case["genes"]
    entries = genes * mean
    buckets = 20 ** min(case.get("k", 7), 4) if case["alphabet"] == "aa" else 4 ** min(case.get("k", 13), 9)
    build = entries * (1 + 8 + 4 + 8 + 4 + 4 + 4) + 4 * buckets * case["genomes"] + 16 * genes
    read = entries * 16 + 4 * buckets * case["genomes"] + 4 * genes
    pairs = case["genomes"] * (case["genomes"] - 1) / 2
    hits = pairs * case["genes"] * (2 * 16 + 16 + 12)
    kind = case["kind"]
    if kind == "build":
        total = build
    elif kind == "calls":
        total = 2 * read + 2 * hits
    elif kind == "batch":
        total = sum((build + read) * max(4, case["genomes"] - i) / case["genomes"] +
                    hits * (max(4, case["genomes"] - i) / case["genomes"]) ** 2 for i in range(case["instances"]))
    elif kind == "long":
        total = read + 28 * 2 * case["longest"] + hits
    elif kind == "serve":
        per = (case["arrive_lo"] + case["arrive_hi"]) / 2
        total = case["arrivals"] * (per * mean * 33 + 4 * buckets + read +
                                    case["genomes"] * (2 * 16 * (per + case["genes"]) + 20 * per))
    else:
        total = (build if case.get("build") else 0) + read + hits
    return {"bytes": total, "flops": 0.0}


# -------------------------------------------------------------------- exact

def _table(genome, k, dev="cuda"):
    """Multiplicity vectors and inverted index of a genome, by plain sorts."""
    al, bits = genome.alphabet, BITS[genome.alphabet]
    code_of = torch.zeros(256, dtype=torch.int64, device=dev)
    for i, c in enumerate(LETTERS[al].encode()):
        code_of[c] = i
    sym = code_of[torch.from_numpy(genome.residues).to(dev).long()]
    off = torch.from_numpy(genome.offsets.astype("int64")).to(dev)
    n = off.numel() - 1
    nwin = (off.diff() - k + 1).clamp(min=0)
    gene = torch.arange(n, device=dev).repeat_interleave(nwin)
    at = torch.arange(gene.numel(), device=dev) + (off[:-1] - _offsets(nwin)[:-1]).repeat_interleave(nwin)
    code = torch.zeros_like(at)
    for j in range(k):
        code = (code << bits) | sym[at + j]
    order = torch.argsort(code, stable=True)
    order = order[torch.argsort(gene[order], stable=True)]
    gene, code = gene[order], code[order]
    new = torch.ones_like(gene, dtype=torch.bool)
    new[1:] = (gene[1:] != gene[:-1]) | (code[1:] != code[:-1])
    start = torch.nonzero(new).flatten()
    cnt = torch.diff(start, append=start.new_tensor([gene.numel()]))
    gene, code = gene[start], code[start]
    ix = torch.argsort(code, stable=True)
    return {"n": n, "nwin": nwin, "gene": gene, "code": code, "cnt": cnt, "icode": code[ix], "igene": gene[ix],
            "icnt": cnt[ix], "k": k, "al": al}


def _pad(x, n):
    out = torch.zeros(n, dtype=torch.int64, device=x.device)
    out[: x.numel()] = x
    return out


def _wrap(x, dtype=torch.int32):
    return x.to(torch.int64).to(dtype)


def _exact_dictionary(t, capacity):
    k, bits = t["k"], BITS[t["al"]]
    lead = min(k, LEAD[t["al"]])
    sigma = len(LETTERS[t["al"]])
    bucket = torch.zeros_like(t["icode"])
    for i in range(lead):
        bucket = bucket * sigma + ((t["icode"] >> (bits * (k - 1 - i))) & ((1 << bits) - 1))
    per_gene = torch.bincount(t["gene"], minlength=t["n"])
    per_bucket = torch.bincount(bucket, minlength=sigma ** lead)
    shift = max(1, (t["n"] - 1).bit_length())
    tail_bits = bits * (k - lead)
    if tail_bits + shift <= 32:
        key = ((t["icode"] & ((1 << tail_bits) - 1)) << shift) | t["igene"]
    else:
        key = t["icode"][:0]
    return [_wrap(t["nwin"]), _wrap(_offsets(per_gene)), _pad(t["code"], capacity), _wrap(_pad(t["cnt"], capacity)),
            _wrap(_offsets(per_bucket)), _pad(t["icode"], capacity), _wrap(_pad(t["igene"], capacity)),
            _wrap(_pad(t["icnt"], capacity)), _wrap(_pad(key, capacity))]


def _exact_pair(a, b, filters):
    """Best hits both ways and BBH of two tables: rows, columns, sums of minima and of maxima."""
    lo = torch.searchsorted(b["icode"], a["icode"])
    hi = torch.searchsorted(b["icode"], a["icode"], right=True)
    times = hi - lo
    ia = torch.arange(lo.numel(), device=lo.device).repeat_interleave(times)
    jb = torch.arange(ia.numel(), device=lo.device) + (lo - _offsets(times)[:-1]).repeat_interleave(times)
    pair, inv = torch.unique(a["igene"][ia] * b["n"] + b["igene"][jb], return_inverse=True)
    ca, cb = a["icnt"][ia], b["icnt"][jb]
    m = torch.zeros_like(pair).scatter_add_(0, inv, torch.minimum(ca, cb))
    ga, gb = pair // b["n"], pair % b["n"]
    na, nb = a["nwin"][ga], b["nwin"][gb]
    if filters:
        sa = torch.zeros_like(pair).scatter_add_(0, inv, ca)
        sb = torch.zeros_like(pair).scatter_add_(0, inv, cb)
        k = a["k"]
        la, lb = na + k - 1, nb + k - 1
        keep = (2 * la >= lb) & (2 * lb >= la) & (sa * k >= na) & (sb * k >= nb)
        ga, gb, na, nb, m = ga[keep], gb[keep], na[keep], nb[keep], m[keep]
    d = na + nb - m
    j = m.double() / d.double()
    best_a = torch.zeros(a["n"], dtype=torch.float64, device=j.device).scatter_reduce_(0, ga, j, "amax")
    best_b = torch.zeros(b["n"], dtype=torch.float64, device=j.device).scatter_reduce_(0, gb, j, "amax")
    ab, ba = j == best_a[ga], j == best_b[gb]
    turn = torch.argsort(gb[ba], stable=True)
    sides = [(ga[ab], gb[ab], m[ab], d[ab]), tuple(x[ba][turn] for x in (gb, ga, m, d)),
             tuple(x[ab & ba] for x in (ga, gb, m, d))]
    return sides


def _ptr(rows, n):
    return _offsets(torch.bincount(rows, minlength=n))


def _exact_pairs(groups, filters):
    """CSR best hits and BBH of every pair of every group of tables, in task order."""
    ptr, hits, bptr, both, edges, base = [], [], [], [], [], 0
    for tables in groups:
        bases = [base]
        for t in tables:
            bases.append(bases[-1] + t["n"])
        base = bases[-1]
        for i, j in _pairs(len(tables)):
            a, b = tables[i], tables[j]
            ab, ba, bb = _exact_pair(a, b, filters)
            ptr += [torch.bincount(ab[0], minlength=a["n"]), torch.bincount(ba[0], minlength=b["n"])]
            hits += [ab[1:], ba[1:]]
            bptr.append(torch.bincount(bb[0], minlength=a["n"]))
            both.append(bb)
            edges.append((bases[i] + bb[0], bases[j] + bb[1]))
    bh_rows = sum(x.numel() for x in ptr)
    bbh_rows = sum(x.numel() for x in bptr)
    bh_cap, bbh_cap = 2 * bh_rows + 1024, bbh_rows + 1024
    out = [[_wrap(_offsets(torch.cat(ptr)))] + [_wrap(_pad(torch.cat([h[i] for h in hits]), bh_cap)) for i in range(3)],
           [_wrap(_offsets(torch.cat(bptr)))] + [_wrap(_pad(torch.cat([p[i] for p in both]), bbh_cap)) for i in range(4)]]
    return out, edges, base


def _exact_families(edges, n):
    """Smallest node of each node's component."""
    u, v = torch.cat([e[0] for e in edges]), torch.cat([e[1] for e in edges])
    label = torch.arange(n, device=u.device)
    while True:
        low = torch.minimum(label[u], label[v])
        new = label.scatter_reduce(0, u, low, "amin").scatter_reduce(0, v, low, "amin")
        new = new[new]
        if torch.equal(new, label):
            return _wrap(label)
        label = new


def exact(case, seed):
    kind = case["kind"]
    if kind == "serve":
        return None
    if kind == "batch":
        groups = [[_table(g, k) for g in genomes] for genomes, k in zip(_batch_genomes(case, seed), _batch_ks(case))]
        return _exact_pairs(groups, False)[0]
    _, genomes, _ = _collection(case, seed)
    tables = [_table(g, case["k"]) for g in genomes]
    if kind == "build":
        return [_exact_dictionary(t, g.residues.size + 1) for t, g in zip(tables, genomes)]
    if kind == "calls":
        a, b = tables
        ab, ba, bb = _exact_pair(a, b, False)
        return [_fixed([x.to(torch.int32).cpu().numpy().view(np.uint32) for x in (_ptr(y[0], n), *y[1:])], n)
                for y, n in ((ab, a["n"]), (ba, b["n"]), ((bb[0], *bb), a["n"]))]
    out, edges, n = _exact_pairs([tables], case.get("filters", False))
    if case.get("families"):
        out.append(_exact_families(edges, n))
    return out
