// C-ABI entry points: argument validation, planning, workspace layout and
// error reporting around the gfx950 kernels.
#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <exception>
#include <memory>
#include <new>
#include <unordered_map>
#include <utility>
#include <vector>

#include "internal.hpp"

using namespace pdp;

namespace {

thread_local char g_last_error[512] = "";

int32_t fail(int32_t code, const char *fmt, ...) __attribute__((format(printf, 2, 3)));
int32_t fail(int32_t code, const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_last_error, sizeof(g_last_error), fmt, ap);
    va_end(ap);
    return code;
}

int32_t hip_fail(hipError_t e, const char *what) {
    return fail(PDP_E_HIP, "%s: %s", what, hipGetErrorString(e));
}

int32_t ok() {
    g_last_error[0] = '\0';
    return PDP_OK;
}

}  // namespace

int32_t pdp::api_fail(int32_t code, const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_last_error, sizeof(g_last_error), fmt, ap);
    va_end(ap);
    return code;
}

struct pdp_plan {
    std::vector<DevTask> tasks;
    std::vector<DevTile> tiles;
    std::vector<DevItem> items;
    std::vector<DevLongSeg> long_segs;  // long-gene path: row segments by first row
    std::vector<DevGroupDict> gdicts;   // group path
    std::vector<DevGroupTgt> gtgts;
    std::vector<DevGroupItem> gitems, gitems_wide;
    std::vector<DevGroupTile> gtiles;
    std::vector<uint8_t> tmap;
    std::vector<uint32_t> ab_row, ba_row, bbh_row;
    std::vector<uint32_t> order;  // order[t]: position of caller task t in the task table
    PlanShape shape;
    uint64_t ws_bytes;
    bool persistent = false;
    mutable bool device_ready = false;  // persistent grids and LDS limit set up on the device
    mutable uint32_t join_grid = 0, tile_grid = 0, fallback_grid = 0;
    // measurement hook: event pairs owned by the plan, one per timed launch
    mutable int32_t timer_kernel = -1;
    mutable uint32_t timer_used = 0;
    uint32_t timer_max = 0;
    mutable std::vector<std::pair<hipEvent_t, hipEvent_t>> timer_events;

    void timer_release() const {
        for (auto &e : timer_events) {
            (void)hipEventDestroy(e.first);
            (void)hipEventDestroy(e.second);
        }
        timer_events.clear();
        timer_kernel = -1;
        timer_used = 0;
    }
    ~pdp_plan() { timer_release(); }
};

extern "C" {

uint32_t pdp_abi_version(void) { return PDP_ABI_VERSION; }

const char *pdp_strerror(int32_t code) {
    switch (code) {
    case PDP_OK: return "ok";
    case PDP_E_INVAL: return "invalid argument";
    case PDP_E_KRANGE: return "k out of range for the alphabet (amino acids 1..12, nucleotides 1..31)";
    case PDP_E_WORKSPACE: return "workspace or arena too small";
    case PDP_E_CAPACITY: return "output or scratch capacity too small";
    case PDP_E_ALPHABET: return "letter outside the dictionary's alphabet, or unknown alphabet";
    case PDP_E_HIP: return "HIP runtime error";
    case PDP_E_BUDGET: return "request exceeds the admission budget";
    case PDP_E_LIMIT: return "size beyond a documented limit";
    case PDP_E_UNIMPL: return "not implemented";
    default: return "unknown error";
    }
}

const char *pdp_last_error(void) { return g_last_error; }

int32_t pdp_k_rule(uint64_t total, uint32_t alphabet, int32_t mode, uint32_t *k_out) {
    if (!k_out || alphabet < 2 || (mode != 0 && mode != 1)) return fail(PDP_E_INVAL, "pdp_k_rule: bad argument");
    // Powers are compared in 128-bit integers so no power near 2^64 overflows.
    unsigned __int128 p = 1;
    uint32_t k = 0;
    if (mode == 0) {
        while (p < total) {
            p *= alphabet;
            ++k;
        }
    } else {
        while (p * alphabet <= total) {
            p *= alphabet;
            ++k;
        }
    }
    *k_out = k < 1 ? 1 : k;
    return ok();
}

// ------------------------------------------------------------ dictionary

static int32_t dict_check(uint32_t n_genes, uint64_t n_residues, uint32_t k, uint32_t alphabet) {
    if (!alpha_known(alphabet)) return fail(PDP_E_ALPHABET, "unknown alphabet %u", alphabet);
    const uint32_t kmax = alpha_spec(alphabet).k_max;
    if (k == 0 || k > kmax) return fail(PDP_E_KRANGE, "k = %u outside 1..%u for this alphabet", k, kmax);
    if (n_genes > PDP_MAX_GENES) return fail(PDP_E_LIMIT, "%u genes exceed %u", n_genes, PDP_MAX_GENES);
    if (n_residues >= (1ull << 32)) return fail(PDP_E_LIMIT, "%llu residues exceed 2^32 - 1", (unsigned long long)n_residues);
    return PDP_OK;
}

static uint64_t dict_arena_bytes(uint32_t n_genes, uint64_t n_residues, uint32_t k, uint32_t alphabet) {
    const uint64_t A = 256, cap = n_residues + 1, nb = n_buckets_for(k, alphabet);
    uint64_t s = 0;
    s += align_up(4 * (uint64_t(n_genes) + 1), A);  // nwin
    s += align_up(4 * (uint64_t(n_genes) + 1), A);  // mv_ptr
    s += align_up(8 * cap, A);                      // mv_code
    s += align_up(4 * cap, A);                      // mv_cnt
    s += align_up(4 * (nb + 1), A);                 // ix_dir
    s += align_up(8 * cap, A);                      // ix_code
    s += align_up(4 * cap, A);                      // ix_gene
    s += align_up(4 * cap, A);                      // ix_cnt
    s += align_up(4 * cap, A);                      // ix_key
    s += align_up(sizeof(pdp_status), A);           // status
    return s;
}

int32_t pdp_dict_size(uint32_t n_genes, uint64_t n_residues, uint32_t k, uint32_t alphabet, uint64_t *arena_bytes,
                      uint64_t *ws_bytes) {
    int32_t rc = dict_check(n_genes, n_residues, k, alphabet);
    if (rc) return rc;
    if (arena_bytes) *arena_bytes = dict_arena_bytes(n_genes, n_residues, k, alphabet);
    if (ws_bytes) {
        *ws_bytes = build_ws_bytes(single_build_shape(n_genes, n_residues, k, alphabet));
    }
    return ok();
}

int32_t pdp_dict_bind(void *arena, uint64_t arena_bytes, uint32_t n_genes, uint64_t n_residues, uint32_t k,
                      uint32_t alphabet, uint32_t flags, pdp_dict *out) {
    if (!arena || !out) return fail(PDP_E_INVAL, "pdp_dict_bind: null pointer");
    if (flags & ~PDP_DICT_LONG_GENES) return fail(PDP_E_INVAL, "pdp_dict_bind: unknown flags 0x%x", flags);
    if (reinterpret_cast<uintptr_t>(arena) % 256) return fail(PDP_E_INVAL, "pdp_dict_bind: arena not 256-byte aligned");
    int32_t rc = dict_check(n_genes, n_residues, k, alphabet);
    if (rc) return rc;
    const uint64_t need = dict_arena_bytes(n_genes, n_residues, k, alphabet);
    if (arena_bytes < need) return fail(PDP_E_WORKSPACE, "arena %llu < %llu bytes", (unsigned long long)arena_bytes, (unsigned long long)need);
    const uint64_t A = 256, cap = n_residues + 1, nb = n_buckets_for(k, alphabet);
    char *p = static_cast<char *>(arena);
    auto take = [&](uint64_t bytes) {
        char *q = p;
        p += align_up(bytes, A);
        return q;
    };
    pdp_dict d;
    std::memset(&d, 0, sizeof(d));
    d.n_genes = n_genes;
    d.k = k;
    d.capacity = cap;
    d.n_buckets = static_cast<uint32_t>(nb);
    d.nwin = reinterpret_cast<uint32_t *>(take(4 * (uint64_t(n_genes) + 1)));
    d.mv_ptr = reinterpret_cast<uint32_t *>(take(4 * (uint64_t(n_genes) + 1)));
    d.mv_code = reinterpret_cast<uint64_t *>(take(8 * cap));
    d.mv_cnt = reinterpret_cast<uint32_t *>(take(4 * cap));
    d.ix_dir = reinterpret_cast<uint32_t *>(take(4 * (nb + 1)));
    d.ix_code = reinterpret_cast<uint64_t *>(take(8 * cap));
    d.ix_gene = reinterpret_cast<uint32_t *>(take(4 * cap));
    d.ix_cnt = reinterpret_cast<uint32_t *>(take(4 * cap));
    d.ix_key = reinterpret_cast<uint32_t *>(take(4 * cap));
    d.key_shift = key_shift_for(n_genes, k, alphabet);
    d.alphabet = alphabet;
    d.lead = lead_letters(k, alphabet);
    d.flags = flags;
    d.status = reinterpret_cast<pdp_status *>(take(sizeof(pdp_status)));
    *out = d;
    return ok();
}

static int32_t build_check(const pdp_genome *genomes, pdp_dict *const *dicts, uint32_t n) {
    if (n == 0 || !genomes || !dicts) return fail(PDP_E_INVAL, "dictionary build: no genomes");
    uint64_t genes = 0, buckets = 0;
    for (uint32_t i = 0; i < n; ++i) {
        const pdp_genome *g = &genomes[i];
        const pdp_dict *d = dicts[i];
        if (!d) return fail(PDP_E_INVAL, "dictionary %u is null", i);
        if (!g->gene_off || (g->n_residues && !g->residues)) return fail(PDP_E_INVAL, "genome %u: null arrays", i);
        int32_t rc = dict_check(g->n_genes, g->n_residues, d->k, d->alphabet);
        if (!rc && (d->lead != lead_letters(d->k, d->alphabet) || d->n_buckets != n_buckets_for(d->k, d->alphabet) ||
                    (d->flags & ~PDP_DICT_LONG_GENES)))
            rc = fail(PDP_E_INVAL, "dictionary %u: fields changed since pdp_dict_bind", i);
        if (rc) return rc;
        if (g->n_genes != d->n_genes || g->n_residues + 1 > d->capacity)
            return fail(PDP_E_INVAL, "genome %u (%u genes, %llu residues) does not match its dictionary (%u genes, capacity %llu)",
                        i, g->n_genes, (unsigned long long)g->n_residues, d->n_genes, (unsigned long long)d->capacity);
        genes += g->n_genes;
        buckets += d->n_buckets;
    }
    if (genes >= UINT32_MAX || buckets >= UINT32_MAX) return fail(PDP_E_LIMIT, "build too large for 32-bit indices");
    return PDP_OK;
}

int32_t pdp_dict_build_many_ws_size(const pdp_genome *genomes, pdp_dict *const *dicts, uint32_t n, uint64_t *ws_bytes) {
    if (!ws_bytes) return fail(PDP_E_INVAL, "pdp_dict_build_many_ws_size: null output");
    int32_t rc = build_check(genomes, dicts, n);
    if (rc) return rc;
    *ws_bytes = build_ws_bytes(build_shape(genomes, dicts, n));
    return ok();
}

int32_t pdp_dict_build_many(const pdp_genome *genomes, pdp_dict *const *dicts, uint32_t n, void *ws, uint64_t ws_bytes,
                            void *stream) {
    if (!ws) return fail(PDP_E_INVAL, "dictionary build: null workspace");
    int32_t rc = build_check(genomes, dicts, n);
    if (rc) return rc;
    const uint64_t need = build_ws_bytes(build_shape(genomes, dicts, n));
    if (ws_bytes < need) return fail(PDP_E_WORKSPACE, "workspace %llu < %llu bytes", (unsigned long long)ws_bytes, (unsigned long long)need);
    hipError_t e = launch_dict_build_many(genomes, dicts, n, ws, static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return hip_fail(e, "dictionary build");
    return ok();
}

int32_t pdp_dict_build(const pdp_genome *g, pdp_dict *d, void *ws, uint64_t ws_bytes, void *stream) {
    if (!g || !d) return fail(PDP_E_INVAL, "pdp_dict_build: null pointer");
    return pdp_dict_build_many(g, &d, 1, ws, ws_bytes, stream);
}

// ------------------------------------------------------------------ plans

static DevDict dev_dict(const pdp_dict *d) {
    DevDict x;
    x.ix_code = d->ix_code;
    x.ix_gene = d->ix_gene;
    x.ix_cnt = d->ix_cnt;
    x.ix_dir = d->ix_dir;
    x.nwin = d->nwin;
    x.ix_key = d->ix_key;
    x.mv_ptr = d->mv_ptr;
    x.mv_code = d->mv_code;
    x.mv_cnt = d->mv_cnt;
    x.n_genes = d->n_genes;
    x.n_buckets = d->n_buckets;
    x.k = d->k;
    x.key_shift = d->key_shift;
    x.bits = alpha_spec(d->alphabet).bits;
    x.lead = d->lead;
    return x;
}

// Records expected in one direction of a task: divergent homologs share a fraction of their k-mers;
// an eighth of the entries per direction covers the family workloads with room; more needs a
// capacity retry.
static uint64_t direction_estimate(const pdp_task &t) { return (t.a->capacity + t.b->capacity) / 8 + 4096; }
// Default tile height of a direction with rows of R: rows of long genes (over 512 letters on average,
// e.g. nucleotide genes) go 32 to a tile.
static uint32_t default_shift(const pdp_dict *R) {
    return R->n_genes && R->capacity / R->n_genes > 512 ? kDefaultTileShift - 1 : kDefaultTileShift;
}
// Records expected of a direction whose tiles are `lower` halvings below their default height, with room:
// the fewer rows, the further their lengths and their share lie from the average (a region that overflows
// costs the two-pass join: two genomes of 1001 genes, tiles of 4 rows, 37 us of 90).
static uint64_t with_slack(uint64_t dir_est, uint32_t lower) { return dir_est * (4 + 3 * uint64_t(lower)) / 4; }
// Records of a direction, slack included, up to which its tiles may go lower by default: 16 MiB of
// them, so that with its other tables (under 512 tiles) no plan of one direction comes near the 64 MiB
// of pdp_bh_noalloc by it.  Two genomes of 5000 genes expect 0.4 million.
constexpr uint64_t kLowTileRecords = 1u << 21;

// Code of the first k-mer of bucket b.
static uint64_t bucket_code(const pdp_dict *d, uint64_t b) {
    const AlphaSpec a = alpha_spec(d->alphabet);
    uint64_t c = 0;
    for (uint32_t i = 0; i < d->lead; ++i) {
        c |= (b % a.sigma) << (a.bits * i);
        b /= a.sigma;
    }
    return c << (a.bits * (d->k - d->lead));
}

// The group path's share of a plan: which tasks take it, and their tables (in_group[t] is set).  A
// group is a connected component of the task graph, with at least a quarter of its pairs compared,
// whose pair-by-pair join would search its entries often enough (gain: searched entries by those the
// group path reads, (D - 1) / 2 for all pairs of D genomes), and whose k-mers meet at most kGroupChance
// k-mers of a target genome by chance.  The gain that pays falls with the group's size, whose passes fill
// the chip, and with filters, which cost the pair path more.  Launch times without the builds, pair path
// against group path, k = 6, even letters; in brackets with filters:
//   1000 genes: 8 genomes (3.5) 107 / 136 [107 / 116], 10 (4.5) 138 / 159 [150 / 137], 12 (5.5) 178 / 173 [199 / 157]
//   2000 genes: 6 (2.5) 110 / 149 [114 / 130], 8 (3.5) 158 / 186 [174 / 160], 10 (4.5) 222 / 223 [244 / 196]
//   4000 genes: 6 (2.5) 180 / 215 [194 / 187], 8 (3.5) 297 / 288 [311 / 256], 10 (4.5) 466 / 400 [503 / 359]
// with the letters of proteins 8 x 4000 553 / 522, near-identical genomes 883 / 713, 1333 nucleotide genes
// 243 / 215.  Under a million entries both take mostly launches (9 x 300 genes 81 / 89 us [89 / 75]).
// Every chance match costs a descriptor, whatever the pair path spends on it: 12 x 1000 genes, k = 5 (0.1
// by chance) 329 / 375 us, k = 6 (0.005) 170 / 155; 10 x 3000 nucleotide genes, k = 13 (0.045) 811 / 750.
constexpr uint64_t kGroupSmall = 1000000;      // entries of a plan up to which a gain of kGroupGain is enough
constexpr double kGroupGain = 2.6, kGroupGainFilt = 1.8;
constexpr double kGroupFixed = 7e6, kGroupFixedFilt = 4e6;  // searched entries past that which a larger plan has to save
constexpr double kGroupChance = 0.05;  // expected chance matches per k-mer and target genome, at most
static uint64_t plan_groups(pdp_plan *P, const pdp_task *tasks, uint32_t n_tasks, const std::vector<uint8_t> &is_long,
                            bool filt, std::vector<uint8_t> &in_group) {
    std::vector<const pdp_dict *> dicts;
    std::vector<uint32_t> ta(n_tasks, UINT32_MAX), tb(n_tasks, UINT32_MAX);
    {
        std::unordered_map<const void *, uint32_t> index;
        auto id = [&](const pdp_dict *d) {
            auto r = index.emplace(d->ix_dir, static_cast<uint32_t>(dicts.size()));
            if (r.second) dicts.push_back(d);
            return r.first->second;
        };
        for (uint32_t t = 0; t < n_tasks; ++t)
            if (!is_long[t]) {
                ta[t] = id(tasks[t].a);
                tb[t] = id(tasks[t].b);
            }
    }
    const uint32_t nd = static_cast<uint32_t>(dicts.size());
    std::vector<uint32_t> root(nd);
    for (uint32_t i = 0; i < nd; ++i) root[i] = i;
    auto find = [&](uint32_t x) {
        while (root[x] != x) x = root[x] = root[root[x]];
        return x;
    };
    for (uint32_t t = 0; t < n_tasks; ++t)
        if (ta[t] != UINT32_MAX) root[find(ta[t])] = find(tb[t]);
    std::vector<uint32_t> comp(nd), local(nd);  // component of each dictionary and its place there
    std::vector<std::vector<uint32_t>> members, ctasks;
    std::vector<uint32_t> of_root(nd, UINT32_MAX);
    for (uint32_t i = 0; i < nd; ++i) {
        uint32_t &c = of_root[find(i)];
        if (c == UINT32_MAX) {
            c = static_cast<uint32_t>(members.size());
            members.emplace_back();
            ctasks.emplace_back();
        }
        comp[i] = c;
        local[i] = static_cast<uint32_t>(members[c].size());
        members[c].push_back(i);
    }
    for (uint32_t t = 0; t < n_tasks; ++t)
        if (ta[t] != UINT32_MAX) ctasks[comp[ta[t]]].push_back(t);
    uint64_t entries = 0, all_rows = 0, all_cap = 0;
    for (uint32_t t = 0; t < n_tasks; ++t)
        if (ta[t] != UINT32_MAX) all_rows += std::max(tasks[t].a->n_genes, tasks[t].b->n_genes);
    for (const pdp_dict *d : dicts) all_cap += d->capacity;
    // small plans: smaller items and tiles, so that the chip's work-group slots are filled once
    const uint64_t target = std::min<uint64_t>(kGroupTarget, std::max<uint64_t>(256, all_cap / 1024));
    const double fill_rows = std::max(16.0, double(all_rows) / 1536.0);
    struct Run {  // the items of one group: buckets in steps of nb, from every multiple of unit on
        uint32_t dict0, n_dicts, nb, n_buckets, unit;
        bool wide;
    };
    std::vector<Run> runs;
    for (uint32_t c = 0; c < members.size(); ++c) {
        const std::vector<uint32_t> &M = members[c];
        const uint32_t D = static_cast<uint32_t>(M.size());
        if (D < 3 || D > kGroupMaxDicts) continue;
        uint64_t cap = 0, genes = 0, searched = 0;
        for (uint32_t i : M) {
            cap += dicts[i]->capacity;
            genes += dicts[i]->n_genes;
        }
        for (uint32_t t : ctasks[c]) searched += std::min(tasks[t].a->capacity, tasks[t].b->capacity);
        const double share = double(cap) / double(all_cap);  // several groups fill the chip together
        const double pays = all_cap <= kGroupSmall ? kGroupGain * double(cap)
                                                   : (filt ? kGroupGainFilt * double(cap) + kGroupFixedFilt * share
                                                           : kGroupGain * double(cap) + kGroupFixed * share);
        if (double(searched) < pays || ctasks[c].size() * 8 < uint64_t(D) * (D - 1)) continue;
        const pdp_dict *d0 = dicts[M[0]];
        const AlphaSpec al = alpha_spec(d0->alphabet);
        const double per_kmer = std::pow(double(al.sigma), -double(d0->k)) * (double(cap) / D);
        const double chance = per_kmer * (double(cap) / double(std::max<uint64_t>(genes, 1)));  // per gene
        if (per_kmer > kGroupChance || entries + cap >= UINT32_MAX) continue;
        // directed edges: both directions as one edge whose columns give the other's best hits
        std::vector<uint8_t> map(uint64_t(D) * D, 255);
        std::vector<std::vector<DevGroupTgt>> out(D);
        std::vector<uint32_t> deg(D, 0);
        for (uint32_t t : ctasks[c]) {
            ++deg[local[ta[t]]];
            ++deg[local[tb[t]]];
        }
        bool ok = true;
        for (uint32_t t : ctasks[c]) {
            uint32_t s = local[ta[t]], x = local[tb[t]];
            uint32_t row = P->ab_row[t], col = P->ba_row[t];
            const bool both = row != UINT32_MAX && col != UINT32_MAX;
            // rows at the genome with many more comparisons; else at the group's earlier one, so that a
            // source's targets follow it in every run of postings
            const bool turn = both ? deg[x] > 2 * deg[s] || (deg[s] <= 2 * deg[x] && s > x) : row == UINT32_MAX;
            if (turn) {
                std::swap(s, x);
                std::swap(row, col);
            }
            uint8_t &m = map[uint64_t(s) * D + x];
            if (s == x || m != 255 || (both && map[uint64_t(x) * D + s] != 255)) {
                ok = false;  // a genome with itself, or the same comparison twice
                break;
            }
            m = static_cast<uint8_t>(out[s].size());
            const pdp_dict *target = dicts[M[x]];
            out[s].push_back(DevGroupTgt{target->nwin, target->n_genes, row, both ? col : UINT32_MAX, 0});
        }
        if (!ok) continue;
        // items: buckets holding about kGroupTarget entries; a k-mer's identity there is its code's
        // low word when the codes of every item span less than 2^32.  Codes jump where a leading
        // letter changes (5 bits for 20 letters), so items then end at every multiple of `unit`
        // buckets, unit a power of the letters: at most twice the items.  Where that does not do,
        // the whole code is the identity; items of a few buckets instead would keep the narrow one but
        // be mostly empty (10 x 3000 genes, k = 10: 160000 items, 1018 us, 209 so; the
        // pair path 325.  k = 25 nucleotides, 10 x 3000: 262144 items, 1552 us, 353 so; the pair path 615).
        const uint64_t nbk = d0->n_buckets;
        const uint64_t nb = std::min<uint64_t>(nbk, std::max<uint64_t>(1, target * nbk / std::max<uint64_t>(cap, 1)));
        const uint32_t tail = al.bits * (d0->k - d0->lead);
        auto narrow = [&](uint64_t unit) {
            if (al.bits * d0->k <= 32) return true;
            if (tail > 32) return false;
            for (uint64_t u = 0; u < nbk; u += unit)
                for (uint64_t b = u; b < std::min(nbk, u + unit); b += nb) {
                    const uint64_t last = std::min({nbk, u + unit, b + nb}) - 1;
                    if (bucket_code(d0, last) - bucket_code(d0, b) + (1ull << tail) > (1ull << 32)) return false;
                }
            return true;
        };
        uint64_t unit = nbk;
        bool is_narrow = narrow(unit);
        while (!is_narrow && unit / al.sigma >= nb) {
            unit /= al.sigma;
            is_narrow = narrow(unit);
        }
        if (!is_narrow) unit = nbk;
        runs.push_back({static_cast<uint32_t>(P->gdicts.size()), D, static_cast<uint32_t>(nb), static_cast<uint32_t>(nbk),
                        static_cast<uint32_t>(unit), !is_narrow});
        // a tile's rows share one table: fewer rows where rows meet many columns by chance
        const double want = std::min(std::min<double>(kGroupTileRows, fill_rows), 1100.0 / (chance + 2.0));
        for (uint32_t i = 0; i < D; ++i) {
            const pdp_dict *d = dicts[M[i]];
            DevGroupDict g{};
            g.ix_code = d->ix_code;
            g.ix_gene = d->ix_gene;
            g.ix_cnt = d->ix_cnt;
            g.ix_dir = d->ix_dir;
            g.nwin = d->nwin;
            g.mv_ptr = d->mv_ptr;
            g.n_genes = d->n_genes;
            g.n_tgt = static_cast<uint32_t>(out[i].size());
            g.tgt_base = static_cast<uint32_t>(P->gtgts.size());
            g.tmap_base = static_cast<uint32_t>(P->tmap.size());
            g.n_dicts = D;
            g.k = d->k;
            for (uint32_t x = 0; x < i; ++x) g.back |= map[uint64_t(i) * D + x] != 255;
            while ((1ull << P->shape.gene_bits) < d->n_genes) ++P->shape.gene_bits;
            g.tile_base = static_cast<uint32_t>(P->gtiles.size());
            g.desc_base = static_cast<uint32_t>(entries);
            entries += d->capacity;
            while (g.n_tgt && (2u << g.gshift) * g.n_tgt <= want) ++g.gshift;
            if (g.n_tgt)
                for (uint32_t g0 = 0; g0 < d->n_genes; g0 += 1u << g.gshift)
                    P->gtiles.push_back(DevGroupTile{static_cast<uint32_t>(P->gdicts.size()), g0,
                                                     std::min<uint32_t>(1u << g.gshift, d->n_genes - g0), 0});
            P->gtgts.insert(P->gtgts.end(), out[i].begin(), out[i].end());
            P->tmap.insert(P->tmap.end(), map.begin() + uint64_t(i) * D, map.begin() + uint64_t(i + 1) * D);
            P->gdicts.push_back(g);
        }
        P->shape.gmax_dicts = std::max(P->shape.gmax_dicts, D);
        for (uint32_t t : ctasks[c]) in_group[t] = 1;
    }
    // items of all groups by bucket range (as a fraction of the group's buckets)
    std::vector<std::pair<double, DevGroupItem>> order[2];
    for (const Run &r : runs)
        for (uint64_t u = 0; u < r.n_buckets; u += r.unit) {
            const uint64_t end = std::min<uint64_t>(r.n_buckets, u + r.unit);
            for (uint64_t b = u; b < end; b += r.nb)
                order[r.wide].push_back({double(b) / r.n_buckets,
                                         DevGroupItem{r.dict0, r.n_dicts, static_cast<uint32_t>(b),
                                                      static_cast<uint32_t>(std::min<uint64_t>(r.nb, end - b))}});
        }
    for (int w = 0; w < 2; ++w) {
        if (runs.size() > 1)
            std::stable_sort(order[w].begin(), order[w].end(), [](const auto &x, const auto &y) { return x.first < y.first; });
        for (const auto &x : order[w]) (w ? P->gitems_wide : P->gitems).push_back(x.second);
    }
    return entries;
}

static int32_t plan_create(const pdp_task *tasks, uint32_t n_tasks, const pdp_params *params, pdp_plan **out) {
    if (!out || (n_tasks && !tasks)) return fail(PDP_E_INVAL, "pdp_plan_create: null pointer");
    *out = nullptr;
    if (n_tasks == 0) return fail(PDP_E_INVAL, "pdp_plan_create: no tasks");
    pdp_params prm;
    std::memset(&prm, 0, sizeof(prm));
    if (params) prm = *params;
    const uint32_t lds_budget = prm.lds_budget ? prm.lds_budget : kDefaultLdsBudget;
    const uint32_t join_entries = prm.join_entries ? prm.join_entries : kJoinLdsCap / 2;  // ~2x headroom to the stage
    if (lds_budget > kMaxTileLds) return fail(PDP_E_INVAL, "lds_budget above %u bytes", kMaxTileLds);
    if (join_entries > kJoinLdsCap) return fail(PDP_E_INVAL, "join_entries above %u", kJoinLdsCap);
    if (prm.tile_rows > kTileMaxRows) return fail(PDP_E_INVAL, "tile_rows above %u", kTileMaxRows);
    if (prm.inc_capacity > UINT32_MAX) return fail(PDP_E_LIMIT, "record capacity above 2^32 - 1");
    uint32_t base_shift = kDefaultTileShift;  // tile rows: the largest power of two <= tile_rows
    if (prm.tile_rows)
        for (base_shift = 0; (2u << base_shift) <= prm.tile_rows; ++base_shift) {
        }
    if (prm.flags & ~(PDP_PARAM_PERSISTENT | PDP_PARAM_COLMAX | PDP_PARAM_TWO_PASS))
        return fail(PDP_E_INVAL, "unknown parameter flags 0x%x", prm.flags);
    if (prm.theta_den && prm.theta_num > prm.theta_den) return fail(PDP_E_INVAL, "theta above 1");
    const bool filt = prm.theta_den || prm.tau_den;

    std::unique_ptr<pdp_plan> owner(new pdp_plan());
    pdp_plan *P = owner.get();
    // Rows of all tasks and directions: short plans take lower tiles, to fill the chip.
    uint64_t all_rows = 0;
    for (uint32_t t = 0; t < n_tasks; ++t)
        if (tasks[t].a && tasks[t].b) {
            const uint32_t f = (tasks[t].flags & PDP_TASK_BBH) ? PDP_TASK_AB | PDP_TASK_BA : tasks[t].flags;
            all_rows += ((f & PDP_TASK_AB) ? tasks[t].a->n_genes : 0u) + ((f & PDP_TASK_BA) ? tasks[t].b->n_genes : 0u);
        }
    // halvings of a direction's tiles below their default height (none where the caller chose it)
    auto lowered = [&](const pdp_dict *R, uint32_t shift) {
        return prm.tile_rows ? 0u : std::max(default_shift(R), shift) - shift;
    };
    // Pass 1, in the caller's order: validation, output row layout, tile height per direction.
    uint64_t bh_rows = 0, bbh_rows = 0;
    // the sorted and hashed tile paths keep 8 bytes per record (12 with the filters' sums)
    uint32_t tile_lds = std::max<uint32_t>(lds_budget, (filt ? 12 : 8) * kTileCap);
    std::vector<DevTask> caller(n_tasks);
    std::vector<uint64_t> cost(n_tasks), task_est(n_tasks, 0);  // join cost, expected records
    std::vector<uint8_t> is_long(n_tasks, 0);  // the task takes the long-gene path
    for (uint32_t t = 0; t < n_tasks; ++t) {
        const pdp_task &tk = tasks[t];
        if (!tk.a || !tk.b) return fail(PDP_E_INVAL, "task %u: null dictionary", t);
        if (tk.a->k != tk.b->k || tk.a->alphabet != tk.b->alphabet || tk.a->lead != tk.b->lead ||
            tk.a->n_buckets != tk.b->n_buckets)
            return fail(PDP_E_INVAL, "task %u: dictionaries built with different k or alphabet (k %u/%u, alphabet %u/%u)",
                        t, tk.a->k, tk.b->k, tk.a->alphabet, tk.b->alphabet);
        uint32_t flags = tk.flags & (PDP_TASK_AB | PDP_TASK_BA | PDP_TASK_BBH);
        if (flags & PDP_TASK_BBH) flags |= PDP_TASK_AB | PDP_TASK_BA;
        if (!flags) return fail(PDP_E_INVAL, "task %u: no output selected", t);
        DevTask &d = caller[t];
        std::memset(&d, 0, sizeof(d));
        const bool long_task = ((tk.a->flags | tk.b->flags) & PDP_DICT_LONG_GENES) != 0;
        is_long[t] = long_task ? 1 : 0;
        // The join searches every entry of its query genome (the task's a) in the other one, so
        // the smaller genome (by entry capacity) takes that side: the task then holds the caller's
        // genomes swapped, with its directions swapped alike (kTaskSwapped); output rows keep the
        // caller's layout.
        const bool swap = !long_task && tk.b->capacity < tk.a->capacity;
        const pdp_dict *qa = swap ? tk.b : tk.a, *qb = swap ? tk.a : tk.b;
        const uint32_t dflags = swap ? (flags & PDP_TASK_BBH) | ((flags & PDP_TASK_AB) ? PDP_TASK_BA : 0u) |
                                           ((flags & PDP_TASK_BA) ? PDP_TASK_AB : 0u)
                                     : flags;
        d.a = dev_dict(qa);
        d.b = dev_dict(qb);
        // column maxima: b's best hits from the AB tiles' columns, records for one direction
        const bool colmax =
            !long_task && (prm.flags & PDP_PARAM_COLMAX) && (flags & PDP_TASK_AB) && (flags & PDP_TASK_BA);
        d.flags = (colmax ? (dflags & ~PDP_TASK_BA) | kTaskColmax : dflags) | (swap ? kTaskSwapped : 0u);
        d.theta_n = prm.theta_num;
        d.theta_d = prm.theta_den;
        d.tau_n = prm.tau_num;
        d.tau_d = prm.tau_den;
        const uint32_t nb = tk.a->n_buckets;
        const uint64_t e_max = std::max<uint64_t>(std::max(tk.a->capacity, tk.b->capacity), 1);
        // sub-ranges of bpw buckets hold ~join_entries entries of the larger genome; an item
        // takes as many sub-ranges as its directory slice (kJoinDirCap buckets) allows
        // packed keys take half the LDS per staged entry: twice the entries per sub-range
        const bool packed = tk.a->key_shift && tk.b->key_shift;
        uint64_t bpw = uint64_t(join_entries) * (packed ? kJoinLdsCapP / kJoinLdsCap : 1) * nb / e_max;
        bpw = std::min<uint64_t>(std::max<uint64_t>(bpw, 1), std::min<uint64_t>(nb, kJoinDirCap));
        const uint64_t subs = std::max<uint64_t>(1, kJoinDirCap / bpw);
        d.bpw = static_cast<uint32_t>(bpw);
        d.subs = static_cast<uint32_t>(subs);
        d.n_chunks = long_task ? 0u : static_cast<uint32_t>((nb + bpw * subs - 1) / (bpw * subs));
        // output rows in the caller's orientation: a's genes (AB), then b's (BA)
        uint32_t orow[2] = {UINT32_MAX, UINT32_MAX};
        for (uint32_t odir = 0; odir < 2; ++odir) {
            if (!(flags & (1u << odir))) continue;
            orow[odir] = static_cast<uint32_t>(bh_rows);
            bh_rows += (odir == 0 ? tk.a : tk.b)->n_genes;
        }
        const uint64_t dir_est = direction_estimate(tk);
        for (uint32_t dir = 0; dir < 2; ++dir) {  // the task's own directions from here on
            d.row_base[dir] = orow[swap ? 1 - dir : dir];
            d.tile_shift[dir] = base_shift;
            d.tiles_n[dir] = 0;
            if (!(dflags & (1u << dir))) continue;
            if ((dir == 1 && colmax) || long_task) continue;  // rows in the output, no tiles and no records of their own
            const pdp_dict *R = dir == 0 ? qa : qb;
            const pdp_dict *C = dir == 0 ? qb : qa;
            // a tile whose records overflow the LDS sort is summed densely: the column genome's
            // window counts (16 bits each) and at least one row of packed 16-bit sums plus its
            // touched-word bitmap must fit
            const uint64_t W = (uint64_t(C->n_genes) + 1) / 2;
            const uint64_t dense = 4 * (((W + 3) & ~3ull) + (filt ? 3 : 1) * W + (W + 31) / 32);
            if (dense > kMaxTileLds)
                return fail(PDP_E_LIMIT, "task %u: %u target genes do not fit an LDS tile", t, C->n_genes);
            tile_lds = std::max<uint32_t>(tile_lds, static_cast<uint32_t>(dense));
            // Unless the caller fixed the height: to fill the chip a plan with under 256 tiles takes
            // lower ones, or under 512 where a tile's records (a row meets columns by chance, `met`) then
            // fit its hash table in one pass, down to 4 rows and up to 128 tiles per direction (two
            // genomes of 200 genes, k = 4: four tiles of 64 rows each way take 108 us, tiles of 4 rows
            // 12).  No lower in larger plans: each batch of the join reserves a run in every tile it
            // feeds by a device atomic (12 x 3000 genes, k = 5: 0.81 ms with 64 rows, 1.44 with 16).
            if (!prm.tile_rows && R->n_genes) {
                const double len = double(R->capacity) / R->n_genes;
                const double met = 8.0 + len * double(C->capacity) *
                                             std::pow(double(alpha_spec(R->alphabet).sigma), -double(R->k));
                uint32_t &sh = d.tile_shift[dir];
                sh = default_shift(R);
                while (sh > 2 && (R->n_genes >> (sh - 1)) <= 128 &&
                       with_slack(dir_est, default_shift(R) - (sh - 1)) <= kLowTileRecords &&
                       ((all_rows >> sh) < 256 || ((all_rows >> sh) < 512 && double(1u << (sh - 1)) * met <= kHashMax)))
                    --sh;
            }
            task_est[t] += with_slack(dir_est, lowered(R, d.tile_shift[dir]));
            d.tiles_n[dir] = static_cast<uint32_t>((uint64_t(R->n_genes) + (1u << d.tile_shift[dir]) - 1) >>
                                                   d.tile_shift[dir]);
        }
        // the join keeps one LDS counter per tile of the task: taller tiles when there are too many
        while (d.tiles_n[0] + d.tiles_n[1] > kJoinTileCap) {
            const bool can0 = d.tiles_n[0] && d.tile_shift[0] < 8, can1 = d.tiles_n[1] && d.tile_shift[1] < 8;
            if (!can0 && !can1)
                return fail(PDP_E_LIMIT, "task %u: too many genes for %u tiles of %u rows", t, kJoinTileCap, kTileMaxRows);
            const uint32_t dir = can0 && (!can1 || d.tiles_n[0] >= d.tiles_n[1]) ? 0 : 1;
            ++d.tile_shift[dir];
            const uint32_t nrows = dir == 0 ? qa->n_genes : qb->n_genes;
            d.tiles_n[dir] = static_cast<uint32_t>((uint64_t(nrows) + (1u << d.tile_shift[dir]) - 1) >> d.tile_shift[dir]);
        }
        d.bbh_row_base = static_cast<uint32_t>(bbh_rows);
        if (flags & PDP_TASK_BBH) bbh_rows += tk.a->n_genes;
        cost[t] = tk.a->capacity + tk.b->capacity;
        P->ab_row.push_back(orow[0]);
        P->ba_row.push_back(orow[1]);
        P->bbh_row.push_back((flags & PDP_TASK_BBH) ? d.bbh_row_base : UINT32_MAX);
        if (bh_rows >= UINT32_MAX) return fail(PDP_E_LIMIT, "plan too large for 32-bit indices");
    }
    // Tasks of a group leave the pair path: no join items and no tiles of their own.
    std::memset(&P->shape, 0, sizeof(P->shape));
    std::vector<uint8_t> in_group(n_tasks, 0);
    uint64_t group_est = 0;
    bool pair_colmax = false;
    if (n_tasks >= 3 && !(prm.flags & (PDP_PARAM_PERSISTENT | PDP_PARAM_TWO_PASS))) {
        P->shape.gentries = plan_groups(P, tasks, n_tasks, is_long, filt, in_group);
        for (uint32_t t = 0; t < n_tasks; ++t) {
            if (!in_group[t]) continue;
            DevTask &d = caller[t];
            d.a = dev_dict(tasks[t].a);
            d.b = dev_dict(tasks[t].b);
            d.flags = 0;
            d.n_chunks = 0;
            d.tiles_n[0] = d.tiles_n[1] = 0;
            d.row_base[0] = P->ab_row[t];
            d.row_base[1] = P->ba_row[t];
            group_est += direction_estimate(tasks[t]);
        }
    }
    // The group path keeps no records; its hits (best hits from column maxima, and ties of rows past the
    // slab) count against the capacity instead: each belongs to a pair of genes that share a k-mer,
    // of which the pair path keeps a record per direction at least, or, with PDP_PARAM_COLMAX, one for
    // at most two hits.  So what fits by pairs fits here.
    uint64_t rec_est = 0, pair_est = 0;
    for (uint32_t t = 0; t < n_tasks; ++t) {
        rec_est += task_est[t];
        if (!in_group[t]) pair_est += task_est[t];
        pair_colmax |= !in_group[t] && (caller[t].flags & kTaskColmax) != 0;
    }
    // Pass 2, largest tasks first: join items and tiles are numbered in this order, so work-groups
    // (and the persistent kernels' counters) take the long items early.
    // each tile's expected records, the estimate rec_est sums: a region of the one-pass join each
    std::vector<uint64_t> tile_est;
    {
        uint64_t n_tiles = 0;
        for (const DevTask &d : caller) {
            n_tiles += uint64_t(d.tiles_n[0]) + d.tiles_n[1];
        }
        P->tiles.reserve(n_tiles);
        tile_est.reserve(n_tiles);
    }
    uint32_t join_tiles = 1;
    std::vector<uint32_t> by_cost(n_tasks);
    for (uint32_t t = 0; t < n_tasks; ++t) by_cost[t] = t;
    std::stable_sort(by_cost.begin(), by_cost.end(), [&](uint32_t x, uint32_t y) { return cost[x] > cost[y]; });
    P->order.assign(n_tasks, 0);
    uint64_t chunks = 0, cells = 0, long_rows = 0;
    for (uint32_t i = 0; i < n_tasks; ++i) {
        const uint32_t t = by_cost[i];
        P->order[t] = i;
        DevTask d = caller[t];
        d.chunk_base = static_cast<uint32_t>(chunks);
        chunks += d.n_chunks;
        d.cell_base = static_cast<uint32_t>(cells);
        uint32_t tile_local = 0;
        const uint64_t dir_est = direction_estimate(tasks[t]);
        for (uint32_t dir = 0; dir < 2; ++dir) {
            d.tile_base[dir] = static_cast<uint32_t>(P->tiles.size());
            if (!(d.flags & (1u << dir))) continue;
            if (is_long[t]) {  // the long-gene path: a row segment instead of tiles
                const uint32_t nrows = dir == 0 ? d.a.n_genes : d.b.n_genes;
                if (nrows) P->long_segs.push_back(DevLongSeg{i, dir, static_cast<uint32_t>(long_rows), nrows});
                long_rows += nrows;
                continue;
            }
            const uint32_t nrows = dir == 0 ? d.a.n_genes : d.b.n_genes;
            const uint32_t T = 1u << d.tile_shift[dir];
            const pdp_task &tk = tasks[t];
            const uint32_t lower = lowered((dir == 0) != ((d.flags & kTaskSwapped) != 0) ? tk.a : tk.b, d.tile_shift[dir]);
            for (uint32_t r0 = 0; r0 < nrows; r0 += T, ++tile_local) {
                DevTile tl;
                tl.task = i;
                tl.dir = dir;
                tl.row0 = r0;
                tl.nrows = std::min<uint32_t>(T, nrows - r0);
                tl.rbase = 0;
                tl.rcap = 0;
                P->tiles.push_back(tl);
                // the direction's estimate split by rows (a direction without genes expects none)
                tile_est.push_back(nrows ? with_slack(dir_est, lower) * tl.nrows / nrows : 0);
            }
        }
        join_tiles = std::max(join_tiles, tile_local);
        cells += uint64_t(tile_local) * d.n_chunks;
        if (cells >= UINT32_MAX) return fail(PDP_E_LIMIT, "plan too large for 32-bit record counts");
        P->tasks.push_back(d);
        if (chunks > UINT32_MAX || P->tiles.size() >= UINT32_MAX)
            return fail(PDP_E_LIMIT, "plan too large for 32-bit indices");
    }
    {  // the one-pass join's items: each task's bucket ranges of bpw * subs buckets, ordered by range
       // across tasks (a range's first bucket as a fraction of its task's buckets, in kSteps steps),
       // tasks in processing order within a step, so that the items in flight read the same stretch
       // of each genome's index (see the join kernel's XCD mapping).  A counting sort, generating
       // every item once in its place.
        constexpr uint32_t kSteps = 4096;
        auto step_of = [](uint64_t bl, uint64_t mult) {
            const uint64_t x = static_cast<uint64_t>((static_cast<unsigned __int128>(bl) * mult) >> 32);
            return static_cast<uint32_t>(std::min<uint64_t>(x, kSteps - 1));
        };
        std::vector<uint32_t> start(kSteps + 1, 0);
        std::vector<uint64_t> mult(P->tasks.size());
        for (size_t i = 0; i < P->tasks.size(); ++i) {
            const DevTask &d = P->tasks[i];
            mult[i] = (static_cast<uint64_t>(kSteps) << 32) / std::max<uint32_t>(d.a.n_buckets, 1);
            const uint64_t span = uint64_t(d.bpw) * d.subs;
            for (uint32_t c = 0; c < d.n_chunks; ++c) ++start[step_of(c * span, mult[i]) + 1];
        }
        for (uint32_t b = 0; b < kSteps; ++b) start[b + 1] += start[b];
        P->items.resize(chunks);
        for (size_t i = 0; i < P->tasks.size(); ++i) {
            const DevTask &d = P->tasks[i];
            const uint64_t span = uint64_t(d.bpw) * d.subs;
            for (uint32_t c = 0; c < d.n_chunks; ++c) {
                const uint64_t bl = c * span;
                DevItem &it = P->items[start[step_of(bl, mult[i])]++];
                it.adir = d.a.ix_dir + bl;
                it.bdir = d.b.ix_dir + bl;
                it.task = static_cast<uint32_t>(i);
                it.n_buckets = static_cast<uint32_t>(std::min<uint64_t>(d.a.n_buckets - bl, span));
                it.bl = static_cast<uint32_t>(bl);
                it.reserved = 0;
            }
        }
    }
    P->shape.n_tasks = n_tasks;
    P->shape.n_gdicts = static_cast<uint32_t>(P->gdicts.size());
    P->shape.n_gtgts = static_cast<uint32_t>(P->gtgts.size());
    P->shape.n_gitems = static_cast<uint32_t>(P->gitems.size());
    P->shape.n_gitems_wide = static_cast<uint32_t>(P->gitems_wide.size());
    P->shape.n_gtiles = static_cast<uint32_t>(P->gtiles.size());
    P->shape.n_tmap = static_cast<uint32_t>(P->tmap.size());
    P->shape.theta_n = prm.theta_num;
    P->shape.theta_d = prm.theta_den;
    P->shape.tau_n = prm.tau_num;
    P->shape.tau_d = prm.tau_den;
    P->shape.total_chunks = static_cast<uint32_t>(chunks);
    P->shape.total_tiles = static_cast<uint32_t>(P->tiles.size());
    P->shape.total_cells = static_cast<uint32_t>(cells);
    P->shape.bh_rows = static_cast<uint32_t>(bh_rows);
    P->shape.bbh_rows = static_cast<uint32_t>(bbh_rows);
    P->shape.tile_lds = static_cast<uint32_t>(align_up(tile_lds, 16));
    P->shape.inc_cap = prm.inc_capacity ? prm.inc_capacity : std::min<uint64_t>(rec_est, UINT32_MAX);
    P->shape.rec_cap = prm.inc_capacity ? prm.inc_capacity : std::min<uint64_t>(pair_est, UINT32_MAX);
    P->shape.fused = (prm.flags & PDP_PARAM_TWO_PASS) ? 0u : 1u;
    P->shape.join_tiles = join_tiles;
    P->shape.fallback_grid = 0;
    {  // regions of the one-pass join: the record capacity split in proportion to the estimates
        unsigned __int128 est_sum = 0;
        for (uint64_t e : tile_est) est_sum += e;
        uint64_t at = 0;
        for (size_t ti = 0; ti < P->tiles.size(); ++ti) {
            const uint64_t cap = est_sum ? static_cast<uint64_t>(
                                               static_cast<unsigned __int128>(P->shape.rec_cap) * tile_est[ti] / est_sum)
                                         : 0;
            P->tiles[ti].rbase = static_cast<uint32_t>(at);
            P->tiles[ti].rcap = static_cast<uint32_t>(cap);
            at += cap;
        }
    }
    P->shape.join_grid = 0;
    P->shape.tile_grid = 0;
    P->shape.colmax = pair_colmax || P->shape.n_gdicts ? 1u : 0u;
    P->shape.cand_cap = pair_colmax ? P->shape.rec_cap : 0;
    if (P->shape.n_gdicts) {
        // listed candidates (16 bytes): pairs at a column's running maximum, whose number depends on the order
        // of the tiles; half of one direction's estimate holds some forty a gene and keeps the scratch
        // at the pair path's size (50 genomes of 4000 genes: 5.4 GB, 7.6 by pairs).  Past them the tiles are
        // replayed against the final maxima, and the hits themselves have to fit.
        P->shape.ghit_cap = P->shape.inc_cap * ((prm.flags & PDP_PARAM_COLMAX) ? 2 : 1);
        P->shape.gcand_cap = std::min<uint64_t>({P->shape.ghit_cap, std::max<uint64_t>(group_est / 2, 1), INT32_MAX});
    }
    P->shape.n_long_segs = static_cast<uint32_t>(P->long_segs.size());
    P->shape.long_rows = static_cast<uint32_t>(long_rows);  // at most the best-hit rows, below 2^32
    P->shape.long_lds = (filt ? 3u : 1u) * kLongCols * 4u;
    P->persistent = (prm.flags & PDP_PARAM_PERSISTENT) != 0;
    P->ws_bytes = pair_ws_bytes(P->shape);
    *out = owner.release();
    return ok();
}

int32_t pdp_plan_create(const pdp_task *tasks, uint32_t n_tasks, const pdp_params *params, pdp_plan **out) {
    try {
        return plan_create(tasks, n_tasks, params, out);
    } catch (const std::exception &) {  // the plan's host tables
        return fail(PDP_E_INVAL, "out of host memory");
    }
}

}  // extern "C"

namespace pdp {
bool plan_all_grouped(const pdp_plan *P) { return P->shape.n_gdicts && !P->shape.total_chunks && !P->shape.long_rows; }

int32_t plan_rebind(pdp_plan *P, const pdp_dict *from, const pdp_dict *to) {
    if (!P || !from || !to) return PDP_E_INVAL;
    if (from->n_genes != to->n_genes || from->capacity != to->capacity || from->k != to->k ||
        from->alphabet != to->alphabet || from->n_buckets != to->n_buckets || from->key_shift != to->key_shift ||
        from->flags != to->flags || (from->ix_key == nullptr) != (to->ix_key == nullptr))
        return PDP_E_INVAL;
    // served requests compare one genome with all residents, which searches no entry of it often enough for a group
    if (!P->gdicts.empty()) return PDP_E_INVAL;
    const DevDict nd = dev_dict(to);
    const uint32_t *lo = from->ix_dir, *hi = from->ix_dir + from->n_buckets + 1;
    auto move = [&](const uint32_t *p) { return p >= lo && p < hi ? to->ix_dir + (p - lo) : p; };
    for (DevTask &t : P->tasks) {
        if (t.a.ix_dir == from->ix_dir) t.a = nd;
        if (t.b.ix_dir == from->ix_dir) t.b = nd;
    }
    for (DevItem &it : P->items) {
        it.adir = move(it.adir);
        it.bdir = move(it.bdir);
    }
    return PDP_OK;
}
}  // namespace pdp

extern "C" {

int32_t pdp_plan_info_get(const pdp_plan *plan, pdp_plan_info *info) {
    if (!plan || !info) return fail(PDP_E_INVAL, "pdp_plan_info_get: null pointer");
    info->ws_bytes = plan->ws_bytes;
    info->inc_capacity = plan->shape.inc_cap;
    info->bh_rows = plan->shape.bh_rows;
    info->bbh_rows = plan->shape.bbh_rows;
    info->n_tasks = plan->shape.n_tasks;
    info->join_groups = plan->shape.total_chunks + plan->shape.n_gitems + plan->shape.n_gitems_wide;
    info->tiles = plan->shape.total_tiles + plan->shape.n_gtiles;
    info->tile_lds = plan->shape.tile_lds;
    info->long_rows = plan->shape.long_rows;
    info->reserved = 0;
    return ok();
}

int32_t pdp_plan_rows(const pdp_plan *plan, uint32_t t, uint32_t *ab_row, uint32_t *ba_row, uint32_t *bbh_row) {
    if (!plan) return fail(PDP_E_INVAL, "pdp_plan_rows: null plan");
    if (t >= plan->shape.n_tasks) return fail(PDP_E_INVAL, "task %u out of range", t);
    if (ab_row) *ab_row = plan->ab_row[t];
    if (ba_row) *ba_row = plan->ba_row[t];
    if (bbh_row) *bbh_row = plan->bbh_row[t];
    return ok();
}

void pdp_plan_destroy(pdp_plan *plan) { delete plan; }

int32_t pdp_plan_upload(const pdp_plan *plan, void *ws, uint64_t ws_bytes, void *stream) {
    if (!plan || !ws) return fail(PDP_E_INVAL, "pdp_plan_upload: null pointer");
    if (ws_bytes < plan->ws_bytes) return fail(PDP_E_WORKSPACE, "workspace %llu < %llu bytes", (unsigned long long)ws_bytes, (unsigned long long)plan->ws_bytes);
    PairWs w = pair_ws_carve(ws, plan->shape);
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipError_t e = hipMemcpyAsync(w.tasks, plan->tasks.data(), sizeof(DevTask) * plan->tasks.size(), hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return hip_fail(e, "pdp_plan_upload");
    e = hipMemcpyAsync(w.order, plan->order.data(), sizeof(uint32_t) * plan->order.size(), hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return hip_fail(e, "pdp_plan_upload");
    if (!plan->items.empty()) {
        e = hipMemcpyAsync(w.items, plan->items.data(), sizeof(DevItem) * plan->items.size(), hipMemcpyHostToDevice, s);
        if (e != hipSuccess) return hip_fail(e, "pdp_plan_upload");
    }
    if (!plan->tiles.empty()) {
        e = hipMemcpyAsync(w.tiles, plan->tiles.data(), sizeof(DevTile) * plan->tiles.size(), hipMemcpyHostToDevice, s);
        if (e != hipSuccess) return hip_fail(e, "pdp_plan_upload");
    }
    if (!plan->gdicts.empty()) {
        auto put = [&](void *dst, const void *src, uint64_t bytes) {
            if (e == hipSuccess && bytes) e = hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, s);
        };
        put(w.gdicts, plan->gdicts.data(), sizeof(DevGroupDict) * plan->gdicts.size());
        put(w.gtgts, plan->gtgts.data(), sizeof(DevGroupTgt) * plan->gtgts.size());
        put(w.gitems, plan->gitems.data(), sizeof(DevGroupItem) * plan->gitems.size());
        put(w.gitems + plan->gitems.size(), plan->gitems_wide.data(), sizeof(DevGroupItem) * plan->gitems_wide.size());
        put(w.gtiles, plan->gtiles.data(), sizeof(DevGroupTile) * plan->gtiles.size());
        put(w.tmap, plan->tmap.data(), plan->tmap.size());
        if (e != hipSuccess) return hip_fail(e, "pdp_plan_upload");
    }
    if (!plan->long_segs.empty()) {
        e = hipMemcpyAsync(w.long_segs, plan->long_segs.data(), sizeof(DevLongSeg) * plan->long_segs.size(),
                           hipMemcpyHostToDevice, s);
        if (e != hipSuccess) return hip_fail(e, "pdp_plan_upload");
    }
    return ok();
}

static int32_t check_outputs(const pdp_plan *plan, const pdp_bh_out *bh, const pdp_bbh_out *bbh, const pdp_status *st) {
    if (!bh || !st) return fail(PDP_E_INVAL, "null output or status");
    if (bh->n_rows != plan->shape.bh_rows || !bh->ptr || (bh->capacity && (!bh->col || !bh->num || !bh->den)))
        return fail(PDP_E_INVAL, "best-hit output: %u rows given, plan has %u", bh->n_rows, plan->shape.bh_rows);
    if (plan->shape.bbh_rows) {
        if (!bbh) return fail(PDP_E_INVAL, "plan has BBH rows but no BBH output was given");
        if (bbh->n_rows != plan->shape.bbh_rows || !bbh->ptr || (bbh->capacity && (!bbh->a || !bbh->b || !bbh->num || !bbh->den)))
            return fail(PDP_E_INVAL, "BBH output: %u rows given, plan has %u", bbh->n_rows, plan->shape.bbh_rows);
    }
    return PDP_OK;
}

int32_t pdp_plan_launch(const pdp_plan *plan, pdp_bh_out *bh, pdp_bbh_out *bbh, pdp_status *status, void *ws,
                        uint64_t ws_bytes, void *stream) {
    if (!plan || !ws) return fail(PDP_E_INVAL, "pdp_plan_launch: null pointer");
    int32_t rc = check_outputs(plan, bh, bbh, status);
    if (rc) return rc;
    if (ws_bytes < plan->ws_bytes) return fail(PDP_E_WORKSPACE, "workspace %llu < %llu bytes", (unsigned long long)ws_bytes, (unsigned long long)plan->ws_bytes);
    PairWs w = pair_ws_carve(ws, plan->shape);
    PlanShape shape = plan->shape;
    if (!plan->device_ready) {
        hipError_t e = allow_tile_lds(plan->shape.tile_lds);
        if (e == hipSuccess && plan->shape.n_gtiles) e = allow_group_lds();
        if (e != hipSuccess) return hip_fail(e, "pdp_plan_launch");
        if (plan->persistent) {
            plan->join_grid = plan->shape.fused ? persistent_fused_grid(plan->shape.join_tiles) : persistent_join_grid();
            plan->tile_grid = persistent_tile_grid(plan->shape.tile_lds);
        }
        if (plan->shape.fused) plan->fallback_grid = persistent_join_grid();
        plan->device_ready = true;
    }
    shape.join_grid = plan->join_grid;
    shape.tile_grid = plan->tile_grid;
    shape.fallback_grid = plan->fallback_grid;
    KernelTimer timer{-1, nullptr, nullptr};
    if (plan->timer_kernel == PDP_KERNEL_BUCKET) {  // no kernel of its own
        if (plan->timer_used < plan->timer_max) plan->timer_used++;
    } else if (plan->timer_kernel >= 0 && plan->timer_used < plan->timer_events.size()) {
        timer.kernel = plan->timer_kernel;
        timer.start = plan->timer_events[plan->timer_used].first;
        timer.stop = plan->timer_events[plan->timer_used].second;
        plan->timer_used++;
    }
    hipError_t e = launch_pairs(shape, w, bh, plan->shape.bbh_rows ? bbh : nullptr, status,
                                static_cast<hipStream_t>(stream), timer.kernel >= 0 ? &timer : nullptr);
    if (e != hipSuccess) return hip_fail(e, "pdp_plan_launch");
    return ok();
}

int32_t pdp_plan_families(const pdp_plan *plan, const pdp_bbh_out *bbh, const uint32_t *node_a, const uint32_t *node_b,
                          uint32_t n_nodes, uint32_t *labels, pdp_status *status, void *ws, uint64_t ws_bytes,
                          void *stream) {
    if (!plan || !bbh || !ws || !status || (n_nodes && (!labels || !node_a || !node_b)))
        return fail(PDP_E_INVAL, "pdp_plan_families: null pointer");
    if (bbh->n_rows != plan->shape.bbh_rows || !bbh->ptr || (bbh->capacity && (!bbh->a || !bbh->b)))
        return fail(PDP_E_INVAL, "pdp_plan_families: BBH output has %u rows, plan has %u", bbh->n_rows,
                    plan->shape.bbh_rows);
    if (ws_bytes < plan->ws_bytes) return fail(PDP_E_WORKSPACE, "workspace %llu < %llu bytes", (unsigned long long)ws_bytes, (unsigned long long)plan->ws_bytes);
    PairWs w = pair_ws_carve(ws, plan->shape);
    hipError_t e = launch_families(plan->shape, w, bbh, node_a, node_b, n_nodes, labels, status,
                                   static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return hip_fail(e, "pdp_plan_families");
    return ok();
}

int32_t pdp_plan_timer_start(pdp_plan *plan, int32_t kernel, uint32_t max_launches) {
    if (!plan || kernel < PDP_KERNEL_JOIN || kernel > PDP_KERNEL_JOIN_BACKUP || max_launches == 0)
        return fail(PDP_E_INVAL, "pdp_plan_timer_start: bad argument");
    plan->timer_release();
    for (uint32_t i = 0; kernel != PDP_KERNEL_BUCKET && i < max_launches; ++i) {
        hipEvent_t a, b;
        hipError_t e = hipEventCreate(&a);
        if (e != hipSuccess) return hip_fail(e, "pdp_plan_timer_start");
        e = hipEventCreate(&b);
        if (e != hipSuccess) {
            (void)hipEventDestroy(a);
            return hip_fail(e, "pdp_plan_timer_start");
        }
        plan->timer_events.emplace_back(a, b);
    }
    plan->timer_kernel = kernel;
    plan->timer_used = 0;
    plan->timer_max = max_launches;
    return ok();
}

int32_t pdp_plan_timer_read(pdp_plan *plan, double *total_ms, uint32_t *launches) {
    if (!plan || !total_ms || !launches) return fail(PDP_E_INVAL, "pdp_plan_timer_read: null pointer");
    double sum = 0;
    for (uint32_t i = 0; i < std::min<size_t>(plan->timer_used, plan->timer_events.size()); ++i) {
        hipError_t e = hipEventSynchronize(plan->timer_events[i].second);
        if (e != hipSuccess) return hip_fail(e, "pdp_plan_timer_read");
        float ms = 0;
        e = hipEventElapsedTime(&ms, plan->timer_events[i].first, plan->timer_events[i].second);
        if (e != hipSuccess) return hip_fail(e, "pdp_plan_timer_read");
        sum += ms;
    }
    *total_ms = sum;
    *launches = plan->timer_used;
    return ok();
}

int32_t pdp_plan_timer_stop(pdp_plan *plan) {
    if (!plan) return fail(PDP_E_INVAL, "pdp_plan_timer_stop: null plan");
    plan->timer_release();
    return ok();
}

int32_t pdp_plan_run(const pdp_plan *plan, pdp_bh_out *bh, pdp_bbh_out *bbh, pdp_status *status, void *ws, uint64_t ws_bytes,
                     void *stream) {
    int32_t rc = pdp_plan_upload(plan, ws, ws_bytes, stream);
    if (rc) return rc;
    return pdp_plan_launch(plan, bh, bbh, status, ws, ws_bytes, stream);
}

// ------------------------------------------------------- single-task forms

int32_t pdp_bh_ws_size(const pdp_dict *q, const pdp_dict *t, const pdp_params *params, uint64_t *ws_bytes) {
    if (!ws_bytes) return fail(PDP_E_INVAL, "pdp_bh_ws_size: null output");
    pdp_task task = {q, t, PDP_TASK_AB, 0};
    pdp_plan *P = nullptr;
    int32_t rc = pdp_plan_create(&task, 1, params, &P);
    if (rc) return rc;
    *ws_bytes = P->ws_bytes;
    delete P;
    return ok();
}

int32_t pdp_bh(const pdp_dict *q, const pdp_dict *t, const pdp_params *params, pdp_bh_out *out, pdp_status *status, void *ws,
               uint64_t ws_bytes, void *stream) {
    pdp_task task = {q, t, PDP_TASK_AB, 0};
    pdp_plan *P = nullptr;
    int32_t rc = pdp_plan_create(&task, 1, params, &P);
    if (rc) return rc;
    rc = pdp_plan_upload(P, ws, ws_bytes, stream);
    if (!rc) {
        // the plan's host tables must outlive the copy
        hipError_t e = hipStreamSynchronize(static_cast<hipStream_t>(stream));
        if (e != hipSuccess) rc = hip_fail(e, "pdp_bh");
    }
    if (!rc) rc = pdp_plan_launch(P, out, nullptr, status, ws, ws_bytes, stream);
    delete P;
    return rc;
}

int32_t pdp_bbh_ws_size(uint32_t n_rows, uint64_t *ws_bytes) {
    if (!ws_bytes) return fail(PDP_E_INVAL, "pdp_bbh_ws_size: null output");
    *ws_bytes = align_up(4ull * scan_partials(n_rows), 256);
    return ok();
}

int32_t pdp_bbh(const pdp_bh_out *ab, const pdp_bh_out *ba, pdp_bbh_out *out, pdp_status *status, void *ws, uint64_t ws_bytes,
                void *stream) {
    if (!ab || !ba || !out || !status || !ws) return fail(PDP_E_INVAL, "pdp_bbh: null pointer");
    if (out->n_rows != ab->n_rows) return fail(PDP_E_INVAL, "pdp_bbh: output has %u rows, input %u", out->n_rows, ab->n_rows);
    if (!ab->ptr || !ba->ptr || !out->ptr) return fail(PDP_E_INVAL, "pdp_bbh: null row pointers");
    uint64_t need = 0;
    pdp_bbh_ws_size(ab->n_rows, &need);
    if (ws_bytes < need) return fail(PDP_E_WORKSPACE, "workspace %llu < %llu bytes", (unsigned long long)ws_bytes, (unsigned long long)need);
    hipError_t e = launch_bbh_standalone(ab, ba, out, status, static_cast<uint32_t *>(ws), static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return hip_fail(e, "pdp_bbh");
    return ok();
}

}  // extern "C"
