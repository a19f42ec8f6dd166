// The group path: best hits of many genome pairs of one set of dictionaries from a single pass
// over their indexes.
//
// The pair path (pairs.hip) joins every genome pair on its own, so an index entry is searched in
// each genome its own is compared with.  Where most pairs of a set of D dictionaries are compared
// (all-pairs collections, batches of them), the shared k-mers of all pairs are found together:
//  1. k_group_join: a work-group takes a range of leading-letter buckets of all D indexes and
//     brings the entries of one k-mer together (a counting sort by a hash of the k-mer in LDS).
//     Every k-mer held by at least two dictionaries gets a run of postings (gene, dictionary,
//     multiplicity), ordered by dictionary, and each member with targets in the run one descriptor
//     (the part of the run that holds its targets, its multiplicity) in the list of the tile that
//     holds its gene's best-hit rows.  A run of two needs no postings: the descriptor holds the
//     partner itself (inline).  A gene has at most as many descriptors as its multiplicity vector
//     has entries, so lists and postings have bounds known from the dictionaries: no count pass,
//     no capacity error.
//  2. k_group_tile: one work-group per tile of a few genes of one dictionary.  It walks the
//     postings of the genes' descriptors and sums the minima of Eq. jaccard_k per (gene, target
//     dictionary, target gene) in an LDS hash table; then every (gene, target) row gets its exact
//     maximum and ties as in the pair path (Eq. best_hit), and the targets' best hits come from
//     the column maxima (Alg. 3) of the same sums.
// Rows with more than kSlab ties leave through the column candidates' list, which counts and
// orders them (k_group_rows, k_group_big; k_colmax_sort).
// Letters are not used evenly, and some k-mers are in many genes: items past the LDS arrays or with a hot
// k-mer go to k_group_join_big, tiles past their hash table to k_group_tile_big.
#include <algorithm>

#include "common.hpp"
#include "internal.hpp"
#include "pair_dev.hpp"

namespace pdp {

constexpr uint32_t kGjThreads = 512;
constexpr uint32_t kGjPer = kGroupCap / kGjThreads;  // entries per thread
constexpr uint32_t kGjSlotBits = 12;
constexpr uint32_t kGjSlots = 1u << kGjSlotBits;     // hash slots of the counting sort, 16 bits each
constexpr uint32_t kGjBigGrid = 512;                 // work-groups for the oversized items: two per CU
constexpr uint32_t kGjMaxPieces = 256;               // pieces an oversized item is listed in
constexpr uint32_t kGjMaxParts = 256;                // hash parts an oversized bucket is cut into
constexpr uint32_t kGjHeatBits = 11;                 // its hash slots, counted to find the hot k-mers
// Entries from which a slot's k-mers are merged one by one: every entry of a slot reads the whole slot (9
// genomes of 2000 genes, a motif in 150 of each: 320 us for its items of 1350 equal k-mers, 74
// with these merged).  Above the
// 255 dictionaries of a group, whose shared genes give runs of one entry each.
constexpr uint32_t kGjHot = 512;
constexpr uint32_t kGjSlotWords = kGjSlots / 2 / kGjThreads;  // words of the slot table a thread scans
using GjMap = uint32_t;  // the dictionaries of a thread's consecutive flat entries, a byte each
static_assert(kGjPer == sizeof(GjMap), "a thread maps its entries as one word");
static_assert(kGroupMaxDicts <= kGjThreads, "one dictionary per thread in the set-up");

// A k-mer's identity inside an item: the low word of its code when the item's codes span less
// than 2^32 (the plan checks it), else the whole code.
template <bool WIDE>
struct GjKey {
    using T = uint32_t;
};
template <>
struct GjKey<true> {
    using T = uint64_t;
};
__device__ __forceinline__ uint32_t gj_mix(uint32_t x) { return x * 2654435761u; }
__device__ __forceinline__ uint32_t gj_mix(uint64_t x) {
    return (static_cast<uint32_t>(x) ^ (static_cast<uint32_t>(x >> 32) * 0x85EBCA6Bu)) * 2654435761u;
}

// An entry in LDS: the k-mer's identity and gene | dictionary << 24, read together.
template <bool WIDE>
struct GjEnt {
    uint32_t key, gd;
};
template <>
struct GjEnt<true> {
    uint64_t key;
    uint32_t gd, pad;
};

template <bool WIDE>
struct alignas(16) GjLds {
    GjEnt<WIDE> ent[kGroupCap];
    uint16_t cnt[kGroupCap];
    uint32_t slot[kGjSlots / 2 + 1];   // two 16-bit counters, then starts, per word
    uint32_t tmp[kGjThreads / kWave + 2];
    uint32_t hot[(1u << kGjHeatBits) / 32];
    uint32_t n, any_hot;
};
// Per dictionary of the group, in dynamic LDS after GjLds.
struct GjDict {
    const uint64_t *code;
    const uint32_t *gene;
    const uint32_t *cnt;
    uint32_t off;        // index entry of the item's flat entry i: off + i
    uint32_t pref;       // flat number of its first entry
    uint32_t tile_base;
    uint32_t src;        // gshift | has targets << 8 | has targets before it << 9
};
constexpr uint32_t kGjLong = 254;    // runs this long keep their length in their postings
constexpr uint32_t kGjInline = 254;  // descriptor length field: the partner itself is in the descriptor

__device__ __forceinline__ uint32_t gj_slot_start(const uint32_t *slot, uint32_t s) {
    return (slot[s >> 1] >> ((s & 1u) * 16u)) & 0xFFFFu;
}

// The dictionary of flat entry i: the last one whose first entry is at or before i.
__device__ __forceinline__ uint32_t gj_dict_of(const GjDict *gd, uint32_t n_dicts, uint32_t i) {
    uint32_t lo = 0, hi = n_dicts;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (gd[mid].pref <= i) lo = mid;
        else hi = mid;
    }
    return lo;
}

// The place of a member's descriptor: a tile's descriptors grow from the front of its part, its
// inline ones from the back.
__device__ __forceinline__ uint32_t gj_desc_slot(const GjDict &d, uint32_t gene, bool inl, uint32_t *__restrict__ cursor) {
    uint32_t *c = cursor + static_cast<uint64_t>(d.tile_base + (gene >> (d.src & 255u))) * kGroupCursorStride;
    return inl ? atomicSub(c + 1, 1u) - 1u : atomicAdd(c, 1u);
}
__device__ __forceinline__ uint32_t gj_row_gene(const GjDict &d, uint32_t gene) {
    return (gene & ((1u << (d.src & 255u)) - 1u)) << 24;
}

// Postings are one word: gene | dictionary << gene_bits | multiplicity above, the largest value of
// whose bits says that the multiplicity is in the low half of the posting's aux word.  The high
// halves of a long run's first two aux words hold its length.
struct GjOut {
    uint32_t *__restrict__ post;
    uint32_t *__restrict__ aux;
    uint2 *__restrict__ desc;
    uint32_t *__restrict__ cursor;
    uint32_t gene_bits;  // at most 24
};

// The posting of a run's member at place pos (the run's len postings begin at start).
__device__ __forceinline__ void gj_post(uint32_t dict, uint32_t gene, uint32_t cnt, uint32_t start, uint32_t len,
                                        uint32_t pos, const GjOut &O) {
    const bool big = len >= kGjLong;
    const uint32_t cb = 24u - O.gene_bits, esc = (1u << cb) - 1u;
    if (cnt >= esc || (big && pos < 2))
        O.aux[start + pos] = cnt | (big ? (pos == 0 ? len << 16 : (pos == 1 ? len & 0xFFFF0000u : 0u)) : 0u);
    O.post[start + pos] = gene | (dict << O.gene_bits) | (cb ? min(cnt, esc) << (O.gene_bits + 8u) : 0u);
}
// A descriptor for the n_t places of the run from place t0 on (a long run's cover all of it).
__device__ __forceinline__ uint2 gj_desc(const GjDict &d, uint32_t gene, uint32_t cnt, uint32_t start, uint32_t len,
                                         uint32_t t0, uint32_t n_t) {
    const bool big = len >= kGjLong;
    return make_uint2(big ? start : start + t0, gj_row_gene(d, gene) | ((big ? 255u : n_t) << 16) | cnt);
}

// The entries in registers (n <= kGroupCap of them, entry q * kGjThreads + tid in slot q) grouped by
// k-mer, runs of at least two dictionaries written out.  False (uniform), with nothing written, when a
// slot holds kGjHot entries or more.  Contains barriers.
template <bool WIDE>
__device__ __forceinline__ bool gj_group(uint32_t n, const typename GjKey<WIDE>::T (&key)[kGjPer],
                                         const uint32_t (&gd)[kGjPer], const uint32_t (&cnt)[kGjPer], GjLds<WIDE> &L,
                                         const GjDict *D, const GjOut &O, uint32_t base) {
    const uint32_t tid = threadIdx.x;
    uint32_t rank[kGjPer];
    if (tid == 0) L.any_hot = 0;
#pragma unroll
    for (uint32_t q = 0; q < kGjPer; ++q) {
        if (q * kGjThreads + tid >= n) continue;
        const uint32_t s = gj_mix(key[q]) >> (32 - kGjSlotBits);
        rank[q] = (atomicAdd(&L.slot[s >> 1], 1u << ((s & 1u) * 16u)) >> ((s & 1u) * 16u)) & 0xFFFFu;
    }
    __syncthreads();
    {  // exclusive scan of the slot sizes
        uint32_t w[kGjSlotWords], sum = 0;
#pragma unroll
        for (uint32_t q = 0; q < kGjSlotWords; ++q) {
            w[q] = L.slot[tid * kGjSlotWords + q];
            sum += (w[q] & 0xFFFFu) + (w[q] >> 16);
            if (max(w[q] & 0xFFFFu, w[q] >> 16) >= kGjHot) L.any_hot = 1;
        }
        uint32_t all;
        uint32_t run = block_exclusive_scan<kGjThreads>(sum, L.tmp, &all);
#pragma unroll
        for (uint32_t q = 0; q < kGjSlotWords; ++q) {
            const uint32_t lo = run, hi = run + (w[q] & 0xFFFFu);
            L.slot[tid * kGjSlotWords + q] = lo | (hi << 16);
            run = hi + (w[q] >> 16);
        }
        if (tid == 0) L.slot[kGjSlots / 2] = n;
    }
    __syncthreads();
    if (L.any_hot) return false;
#pragma unroll
    for (uint32_t q = 0; q < kGjPer; ++q) {
        if (q * kGjThreads + tid >= n) continue;
        const uint32_t p = gj_slot_start(L.slot, gj_mix(key[q]) >> (32 - kGjSlotBits)) + rank[q];
        GjEnt<WIDE> e;
        e.key = key[q];
        e.gd = gd[q];
        L.ent[p] = e;
        L.cnt[p] = static_cast<uint16_t>(cnt[q]);
    }
    __syncthreads();
    // each entry's run: where it starts among the postings (the keys below its own in the slot come
    // first), its length and the entry's place in it by (dictionary, gene).  A source's targets come
    // after it in the run (or, with bit 9 of src, anywhere in it); the tile skips what is no target.
    // The descriptors' places come from atomics on the tiles' cursors: all of a thread's are in
    // flight before the first descriptor is stored.
    uint32_t at[kGjPer];
    uint2 out[kGjPer];
#pragma unroll
    for (uint32_t q = 0; q < kGjPer; ++q) {
        out[q].y = 0;
        const uint32_t p = q * kGjThreads + tid;
        if (p >= n) continue;
        const GjEnt<WIDE> own = L.ent[p];
        const uint32_t s = gj_mix(own.key) >> (32 - kGjSlotBits);
        const uint32_t a = gj_slot_start(L.slot, s), b = gj_slot_start(L.slot, s + 1);
        if (b - a < 2) continue;
        uint32_t less = 0, len = 0, pos = 0, sum = 0;
        for (uint32_t x = a; x < b; ++x) {
            const GjEnt<WIDE> e = L.ent[x];
            const bool same = e.key == own.key;
            less += e.key < own.key;
            len += same;
            pos += same && e.gd < own.gd;
            sum += same ? x : 0u;
        }
        if (len < 2) continue;
        const uint32_t dict = own.gd >> 24, gene = own.gd & 0xFFFFFFu, cnt = L.cnt[p], mate = sum - p;
        const GjDict &d = D[dict];
        const uint32_t t0 = (d.src >> 9) & 1u ? 0u : pos + 1u;
        uint32_t n_t = (d.src >> 8) & 1u ? len - t0 : 0u;
        const bool inl = len == 2 && cnt < 256u && L.cnt[mate] < 256u;  // no postings: the partner goes inline
        if (inl) {
            const uint32_t m = L.ent[mate].gd;
            if ((m >> 24) == dict) n_t = 0;
            out[q] = make_uint2(m, gj_row_gene(d, gene) | (kGjInline << 16) | (L.cnt[mate] << 8) | cnt);
        } else {
            gj_post(dict, gene, cnt, base + a + less, len, pos, O);
            out[q] = gj_desc(d, gene, cnt, base + a + less, len, t0, n_t);
        }
        if (n_t) at[q] = gj_desc_slot(d, gene, inl, O.cursor);
        else out[q].y = 0;
    }
#pragma unroll
    for (uint32_t q = 0; q < kGjPer; ++q)
        if (out[q].y) O.desc[at[q]] = out[q];  // a multiplicity is at least 1: never zero
    return true;
}

// The item's dictionaries into LDS: everything but its entries' numbers.
__device__ __forceinline__ void gj_dict_load(GjDict &D, const DevGroupDict &d) {
    D.code = d.ix_code;
    D.gene = d.ix_gene;
    D.cnt = d.ix_cnt;
    D.tile_base = d.tile_base;
    D.src = d.gshift | (d.n_tgt ? 256u : 0u) | (d.back ? 512u : 0u);
}

// One item whose entries fit the LDS arrays, without a hot slot; the others are listed for
// k_group_join_big.
// 512 threads with 4 entries each (64 VGPRs) fill the CU's 32 wave slots; 256 threads with 8 kept
// 16-20 waves and took 1.23 ms against 1.16 on 50 genomes of 3000 to 5000 genes (6.8e7 entries).
// There it takes 1.04 ms: reading the entries 0.36 (1.1 GB), sorting and walking them 0.27, postings
// 0.08, descriptors 0.33, of which the cursors' device atomics 0.15 (they pass at 26e9/s, and at a
// sixth of that when 32 tiles' cursors share a line, hence kGroupCursorStride).  The pair path's
// join of the 1225 pairs takes 5.27 ms.
template <bool WIDE>
__global__ __launch_bounds__(kGjThreads, WIDE ? 4 : 8) void k_group_join(const DevGroupDict *__restrict__ dicts,
                                                           const DevGroupItem *__restrict__ items,
                                                           uint2 *__restrict__ big, uint32_t *__restrict__ n_big,
                                                           GjOut O) {
    using Key = typename GjKey<WIDE>::T;
    __shared__ GjLds<WIDE> L;
    extern __shared__ uint64_t gj_dyn[];
    GjDict *D = reinterpret_cast<GjDict *>(gj_dyn);
    const uint32_t tid = threadIdx.x;
    const uint32_t item = xcd_item(blockIdx.x, gridDim.x);
    const DevGroupItem it = items[item];
    uint32_t lo = 0, len = 0;
    if (tid < it.n_dicts) {
        const DevGroupDict &d = dicts[it.dict0 + tid];
        lo = load_global(d.ix_dir + it.b0);
        len = load_global(d.ix_dir + it.b0 + it.nb) - lo;
        gj_dict_load(D[tid], d);
    }
    for (uint32_t i = tid; i <= kGjSlots / 2; i += kGjThreads) L.slot[i] = 0;
    uint8_t *map = reinterpret_cast<uint8_t *>(L.ent);  // the dictionary of each flat entry, until the sort
    GjMap *mapw = reinterpret_cast<GjMap *>(L.ent);
    mapw[tid] = 0;
    uint32_t n;
    const uint32_t pref = block_exclusive_scan<kGjThreads>(len, L.tmp, &n);
    if (tid < it.n_dicts) {
        D[tid].pref = pref;
        D[tid].off = lo - pref;
        if (len && pref < kGroupCap) map[pref] = static_cast<uint8_t>(tid);
    }
    if (n < 2) return;  // uniform
    if (n > kGroupCap) {  // uniform: listed in pieces of as many buckets each, fewer than 4 n / kGroupCap of them
        if (tid == 0) {
            uint32_t pieces = 1;
            while (2 * pieces <= min(it.nb, kGjMaxPieces) && pieces * (kGroupCap / 2) < n) pieces *= 2;
            const uint32_t at = atomicAdd(n_big, pieces);
            for (uint32_t x = 0; x < pieces; ++x) big[at + x] = make_uint2(item, x | (pieces << 16));
        }
        return;
    }
    // the item's postings: as many places as the group's indexes hold entries before it
    uint32_t base;
    (void)block_exclusive_scan<kGjThreads>(lo, L.tmp, &base);
    base += dicts[it.dict0].desc_base;
    __syncthreads();
    Key key[kGjPer];
    uint32_t gd[kGjPer], cnt[kGjPer];
    auto load = [&](uint32_t i, uint32_t d, uint32_t q) {
        const uint32_t e = D[d].off + i;
        if constexpr (WIDE) key[q] = load_global(D[d].code + e);
        else key[q] = load_global(reinterpret_cast<const uint32_t *>(D[d].code + e));
        gd[q] = load_global(D[d].gene + e) | (d << 24);
        cnt[q] = load_global(D[d].cnt + e);
    };
    {  // dictionary ids ascend along the flat entries: a running maximum of the marks fills the map
        const GjMap v = mapw[tid];
        uint32_t m = 0;
#pragma unroll
        for (uint32_t j = 0; j < kGjPer; ++j) m = max(m, (v >> (8 * j)) & 255u);
        uint32_t inc = m;
#pragma unroll
        for (uint32_t o = 1; o < kWave; o <<= 1) {
            const uint32_t y = __shfl_up(inc, o, kWave);
            if (lane_id() >= o) inc = max(inc, y);
        }
        if (lane_id() == kWave - 1) L.tmp[tid / kWave] = inc;
        uint32_t before = __shfl_up(inc, 1, kWave);
        if (lane_id() == 0) before = 0;
        __syncthreads();
        for (uint32_t w = 0; w < tid / kWave; ++w) before = max(before, L.tmp[w]);
        GjMap out = 0;
#pragma unroll
        for (uint32_t j = 0; j < kGjPer; ++j) {
            before = max(before, (v >> (8 * j)) & 255u);
            out |= before << (8 * j);
        }
        mapw[tid] = out;
    }
    __syncthreads();
    uint32_t dd[kGjPer];
#pragma unroll
    for (uint32_t q = 0; q < kGjPer; ++q) dd[q] = map[q * kGjThreads + tid];
#pragma unroll
    for (uint32_t q = 0; q < kGjPer; ++q) {
        const uint32_t i = q * kGjThreads + tid;
        if (i < n) load(i, dd[q], q);
    }
    __syncthreads();  // the map's words take the sorted entries
    if (!gj_group<WIDE>(n, key, gd, cnt, L, D, O, base) && tid == 0) big[atomicAdd(n_big, 1u)] = make_uint2(item, 1u << 16);
}

// Pieces of the items past the LDS arrays (letters are not used evenly, so there are some), in ranges of
// buckets that fit.  A single bucket past the arrays is taken in parts by a hash of the k-mer; k-mers in many genes
// of many genomes (motifs, repeats), found by their hash slots' counts, are left out of the parts and
// merged one at a time from the indexes, which are sorted by k-mer.  A kernel of its own: in
// k_group_join its registers cost every item 7% (50 x 4000 genes, uniform letters, 4.63 -> 4.98 ms).
template <bool WIDE>
__global__ __launch_bounds__(kGjThreads, 4) void k_group_join_big(const DevGroupDict *__restrict__ dicts,
                                                                  const DevGroupItem *__restrict__ items,
                                                                  const uint2 *__restrict__ big,
                                                                  const uint32_t *__restrict__ n_big, GjOut O) {
    using Key = typename GjKey<WIDE>::T;
    __shared__ GjLds<WIDE> L;
    extern __shared__ uint64_t gj_dyn[];
    GjDict *D = reinterpret_cast<GjDict *>(gj_dyn);
    const uint32_t tid = threadIdx.x, n_items = *n_big;
    uint32_t lo = 0, len = 0, base = 0;
    uint32_t n_dicts = 0;
    auto key_of = [&](uint32_t d, uint32_t e) {
        if constexpr (WIDE) return load_global(D[d].code + e);
        else return load_global(reinterpret_cast<const uint32_t *>(D[d].code + e));
    };
    // parts go by the hash bits below the heat slot's
    uint32_t parts = 1;
    auto part_of = [&](Key k) { return (gj_mix(k) >> 8) & (parts - 1u); };
    auto heat_of = [&](Key k) { return gj_mix(k) >> (32 - kGjHeatBits); };
    auto is_hot = [&](Key k) { return (L.hot[heat_of(k) >> 5] >> (heat_of(k) & 31u)) & 1u; };
    // the k-mers of the range that `take` accepts, one at a time: thread d walks dictionary d's entries [at, end),
    // the smallest code among the heads is the next k-mer.  Ends with a barrier.
    auto merge = [&](uint32_t at, uint32_t end, auto take) {
        unsigned long long *head_min = reinterpret_cast<unsigned long long *>(L.slot);  // [0]: smallest head
        for (;;) {
            __syncthreads();
            if (tid == 0) {
                head_min[0] = ~0ull;
                L.n = 0;
            }
            __syncthreads();
            uint64_t head = ~0ull;
            for (; at < end; ++at) {
                head = load_global(D[tid].code + at);
                if (take(static_cast<Key>(head))) break;
                head = ~0ull;
            }
            if (at < end) atomicMin(&head_min[0], static_cast<unsigned long long>(head));
            __syncthreads();
            const uint64_t code = head_min[0];
            if (code == ~0ull) break;  // uniform: every index is used up (codes stay below 2^62)
            uint32_t mine = 0;
            if (head == code) {  // the k-mer's run ends before hi
                uint32_t l = at + 1, hi = end;
                for (uint32_t step = 1; l + step <= end; step <<= 1) {
                    if (load_global(D[tid].code + l + step - 1) != code) {
                        hi = l + step - 1;
                        break;
                    }
                    l += step;
                }
                while (l < hi) {
                    const uint32_t mid = (l + hi) >> 1;
                    if (load_global(D[tid].code + mid) == code) l = mid + 1;
                    else hi = mid;
                }
                mine = l - at;
                atomicAdd(&L.n, 1u);
            }
            uint32_t total;
            const uint32_t first = block_exclusive_scan<kGjThreads>(mine, L.tmp, &total);  // contains barriers
            const bool live = L.n > 1;  // uniform
            if (tid < n_dicts) {  // D[].pref / off now number this k-mer's members, by dictionary
                D[tid].pref = first;
                D[tid].off = at - first;
            }
            __syncthreads();
            if (live)
                for (uint32_t i = tid; i < total; i += kGjThreads) {
                    const uint32_t d = gj_dict_of(D, n_dicts, i), e = D[d].off + i;
                    const uint32_t t0 = (D[d].src >> 9) & 1u ? 0u : i + 1u;
                    const uint32_t n_t = (D[d].src >> 8) & 1u ? total - t0 : 0u;
                    const uint32_t gene = load_global(D[d].gene + e), c = load_global(D[d].cnt + e);
                    gj_post(d, gene, c, base, total, i, O);
                    if (n_t) O.desc[gj_desc_slot(D[d], gene, false, O.cursor)] = gj_desc(D[d], gene, c, base, total, t0, n_t);
                }
            at += mine;
            base += total;
        }
        __syncthreads();
    };
    for (uint32_t x = blockIdx.x; x < n_items; x += gridDim.x) {  // uniform
        const uint2 piece = big[x];
        DevGroupItem it = items[piece.x];
        const uint32_t pieces = piece.y >> 16, p0 = it.nb * (piece.y & 0xFFFFu) / pieces;
        it.nb = it.nb * ((piece.y & 0xFFFFu) + 1) / pieces - p0;  // nb * 256 fits 32 bits
        it.b0 += p0;
        n_dicts = it.n_dicts;
        __syncthreads();
        lo = 0;
        if (tid < n_dicts) {
            const DevGroupDict &d = dicts[it.dict0 + tid];
            lo = load_global(d.ix_dir + it.b0);
            gj_dict_load(D[tid], d);
        }
        // the piece's postings: as many places as the group's indexes hold entries before it
        (void)block_exclusive_scan<kGjThreads>(lo, L.tmp, &base);
        base += dicts[it.dict0].desc_base;
        uint32_t width = it.nb;
        for (uint32_t b = 0; b < it.nb; b += width, width = min(2 * width, it.nb - b)) {  // uniform
            // the widest range from bucket b on that fits, halving
            uint32_t m, first;
            for (;; width >>= 1) {
                lo = len = 0;
                if (tid < n_dicts) {
                    const uint32_t *dir = dicts[it.dict0 + tid].ix_dir + it.b0 + b;
                    lo = load_global(dir);
                    len = load_global(dir + width) - lo;
                }
                first = block_exclusive_scan<kGjThreads>(len, L.tmp, &m);
                if (m <= kGroupCap || width == 1) break;  // uniform
            }
            if (m < 2) {
                base += m;
                continue;
            }
            auto number = [&] {  // D[].pref / off number the range's entries, by dictionary
                __syncthreads();
                if (tid < n_dicts) {
                    D[tid].pref = first;
                    D[tid].off = lo - first;
                }
                __syncthreads();
            };
            parts = 1;
            bool any_hot = false, counted = false;
            auto find_hot = [&] {
                number();
                for (uint32_t i = tid; i < (1u << kGjHeatBits); i += kGjThreads) L.slot[i] = 0;
                if (tid == 0) L.n = 0;
                __syncthreads();
                for (uint32_t i = tid; i < m; i += kGjThreads) {
                    const uint32_t d = gj_dict_of(D, n_dicts, i);
                    atomicAdd(&L.slot[heat_of(key_of(d, D[d].off + i))], 1u);
                }
                __syncthreads();
                for (uint32_t w0 = tid; w0 < (1u << kGjHeatBits); w0 += kGjThreads) {  // a wave's 64 slots: two words
                    const uint32_t c = L.slot[w0];
                    const uint64_t hot = __ballot(c >= kGjHot);
                    if ((tid & 31u) == 0) L.hot[w0 >> 5] = static_cast<uint32_t>(hot >> (tid & 32u));
                    if (c >= kGjHot) atomicAdd(&L.n, c);
                }
                __syncthreads();
                any_hot = L.n != 0;
                counted = true;
                const uint32_t rest = m - L.n;
                while (parts < kGjMaxParts && parts * (kGroupCap / 2) < rest) parts <<= 1;
            };
            if (m > kGroupCap) find_hot();
            for (uint32_t p = 0; p < parts; ++p) {
                number();
                for (uint32_t i = tid; i <= kGjSlots / 2; i += kGjThreads) L.slot[i] = 0;
                if (tid == 0) L.n = 0;
                __syncthreads();
                for (uint32_t i = tid; i < m; i += kGjThreads) {
                    const uint32_t d = gj_dict_of(D, n_dicts, i), e = D[d].off + i;
                    const Key k = key_of(d, e);
                    if (counted && (part_of(k) != p || is_hot(k))) continue;
                    const uint32_t at = atomicAdd(&L.n, 1u);
                    if (at >= kGroupCap) continue;
                    L.ent[at].key = k;
                    L.ent[at].gd = load_global(D[d].gene + e) | (d << 24);
                    L.cnt[at] = static_cast<uint16_t>(load_global(D[d].cnt + e));
                }
                __syncthreads();
                const uint32_t got = L.n;
                bool grouped = got <= kGroupCap;  // uniform
                if (grouped) {
                    Key key[kGjPer];
                    uint32_t gd[kGjPer], cnt[kGjPer];
#pragma unroll
                    for (uint32_t q = 0; q < kGjPer; ++q) {
                        const uint32_t i = q * kGjThreads + tid;
                        if (i >= got) continue;
                        key[q] = L.ent[i].key;
                        gd[q] = L.ent[i].gd;
                        cnt[q] = L.cnt[i];
                    }
                    __syncthreads();
                    grouped = gj_group<WIDE>(got, key, gd, cnt, L, D, O, base);
                }
                if (grouped) {
                    base += got;
                } else if (!counted) {  // the one part has a hot slot: again without it
                    find_hot();
                    --p;
                } else {  // too many for the arrays all the same
                    merge(lo, lo + len, [&](Key k) { return part_of(k) == p && !is_hot(k); });
                }
            }
            if (any_hot) merge(lo, lo + len, [&](Key k) { return is_hot(k); });
            __syncthreads();
        }
    }
}

// ------------------------------------------------------------------ tiles

constexpr uint32_t kGtThreads = 256;
constexpr uint32_t kGtThreadsBig = 1024;                  // k_group_tile_big: one work-group per CU,
constexpr uint32_t kGtHashBitsBig = 14;                   // with a table of 2^14 sums (2^13 with filters)
constexpr uint32_t kGtBigGrid = 256;
constexpr uint32_t kGtLongRun = 1024;                     // postings from which a run is taken by all waves
constexpr uint32_t kGtMaxProbe = 48;                      // a longer probe means the table is too full

// A tile kernel's shape: threads, hash table (key and sum per slot, and the occurrences with filters).
template <bool FILT, uint32_t NT_, uint32_t BITS>
struct GtShape {
    static constexpr bool kFilt = FILT;
    static constexpr uint32_t NT = NT_, kBits = BITS, kSlots = 1u << BITS, kPer = kSlots / NT;
    static constexpr uint32_t kWords = (FILT ? 3 : 2) * kSlots;
};
template <bool FILT>
using GtSmall = GtShape<FILT, kGtThreads, kGroupHashBits>;
template <bool FILT>
using GtBig = GtShape<FILT, kGtThreadsBig, kGtHashBitsBig - (FILT ? 1 : 0)>;

template <uint32_t NT>
struct GtLds {
    unsigned long long best[kGroupTileRows];  // row maximum as (m << 32) | d
    const uint32_t *tw[kGroupMaxDicts + 1];   // per target: window counts of its genes
    uint32_t trow[kGroupMaxDicts + 1];        // its best-hit rows for the source's genes
    uint32_t tcol[kGroupMaxDicts + 1];        // its own genes' best-hit rows (column maxima) or UINT32_MAX
    uint32_t tn[kGroupMaxDicts + 1];          // its genes
    uint32_t nr[kGroupTileRows];              // window counts of the tile's genes
    uint32_t ties[kGroupTileRows];            // ties per row; during a walk its long runs
    uint8_t tmap[kGroupMaxDicts + 1];         // group dictionary -> target, 255: none
    uint8_t vr[kGroupTileRows], vt[kGroupTileRows];  // gene and target of each row
    uint8_t mark[NT / kWave][kWave];                 // gt_walk
    unsigned long long cand_base;
    uint32_t over, cand_n, many;
};

// Column maxima of the group's tiles (see ColWs; their candidates may number more than 32 bits hold).
struct GtCols {
    unsigned long long *key;
    uint4 *cands;
    unsigned long long *count;
    uint64_t cap;
};

// A tile's descriptors: [d0, d0 + nd) with postings, [i0, i0 + ni) inline.
struct GtList {
    const uint2 *__restrict__ desc;
    const uint32_t *__restrict__ post;
    const uint32_t *__restrict__ aux;
    uint32_t gene_bits;
    uint32_t d0, nd, i0, ni;
};

// Inclusive maximum over the lanes up to this one (row shifts inside 16 lanes, then the row and
// half-wave broadcasts; every lane active).
__device__ __forceinline__ uint32_t wave_inclusive_max(uint32_t x) {
    auto step = [](uint32_t v, uint32_t o) { return max(v, o); };
    x = step(x, __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, false));
    x = step(x, __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, false));
    x = step(x, __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, false));
    x = step(x, __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, false));
    x = step(x, __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false));
    x = step(x, __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false));
    return x;
}

// Calls f(row gene, its multiplicity, dictionary, gene, multiplicity) for every posting of the
// descriptors of row genes [g0, g1).  Inline descriptors go one per thread.  The others go 64 to a
// wave, their postings laid end to end and taken 64 at a time, so that every lane has one whatever
// the runs' lengths (5.6 postings on average on 50 genomes, up to 49): mark is a wave's 64 bytes
// of LDS, where the descriptors that start inside a window of 64 leave their lane.  The walk ends
// early once S.over is set.  Runs of kGtLongRun postings or more are listed (in S.ties: S.many of them,
// zero before) and taken by all waves together at the end: a tile's lie together, and one wave walked
// them all.  Contains a barrier.
template <uint32_t NT, typename F>
__device__ __forceinline__ void gt_walk(const GtList &T, uint32_t g0, uint32_t g1, GtLds<NT> &S, F f) {
    const volatile uint32_t *stop = &S.over;
    volatile uint8_t *mark = S.mark[threadIdx.x / kWave];
    for (uint32_t i = threadIdx.x; i < T.ni && !*stop; i += NT) {
        const uint2 d = T.desc[T.i0 + i];
        const uint32_t r = d.y >> 24;
        if (r >= g0 && r < g1) f(r, d.y & 255u, d.x >> 24, d.x & 0xFFFFFFu, (d.y >> 8) & 255u);
    }
    const uint32_t lane = lane_id();
    const uint32_t gmask = (1u << T.gene_bits) - 1u, cb = 24u - T.gene_bits, esc = (1u << cb) - 1u;
    auto one = [&](uint32_t y, uint32_t at) {  // posting at of the descriptor with second word y
        const uint32_t p = T.post[at];
        uint32_t c = cb ? p >> (T.gene_bits + 8u) : 0u;
        if (c == esc) c = T.aux[at] & 0xFFFFu;
        f(y >> 24, y & 0xFFFFu, (p >> T.gene_bits) & 255u, p & gmask, c);
    };
    auto long_len = [&](uint32_t start) { return (T.aux[start] >> 16) | (T.aux[start + 1] & 0xFFFF0000u); };
    for (uint32_t base = (threadIdx.x / kWave) * kWave; base < T.nd; base += NT) {
        if (__builtin_amdgcn_readfirstlane(*stop)) break;
        const uint2 d = base + lane < T.nd ? T.desc[T.d0 + base + lane] : make_uint2(0u, 0u);
        const uint32_t r = d.y >> 24;
        uint32_t len = r >= g0 && r < g1 ? (d.y >> 16) & 255u : 0u;
        if (len == 255u) {
            len = long_len(d.x);
            if (len >= kGtLongRun) {
                const uint32_t at = atomicAdd(&S.many, 1u);
                if (at < kGroupTileRows) {
                    S.ties[at] = base + lane;
                    len = 0;
                }
            }
        }
        const uint32_t incl = wave_inclusive_sum(len), first = incl - len;
        const uint32_t total = __shfl(incl, kWave - 1, kWave);
        const uint32_t from = d.x - first;  // flat posting j of this descriptor is post[from + j]
        uint32_t carry = 0;                 // lane + 1 of the descriptor that reaches into the window
        for (uint32_t j = 0; j < total; j += kWave) {
            mark[lane] = 0;
            if (len && first - j < kWave) mark[first - j] = static_cast<uint8_t>(lane + 1);
            const uint32_t own = wave_inclusive_max(max(static_cast<uint32_t>(mark[lane]), lane == 0 ? carry : 0u));
            carry = __builtin_amdgcn_readlane(own, kWave - 1);
            const uint32_t at = __shfl(from, own - 1, kWave) + j + lane, y = __shfl(d.y, own - 1, kWave);
            if (j + lane < total) one(y, at);
        }
    }
    __syncthreads();
    const uint32_t n_long = min(S.many, kGroupTileRows);
    for (uint32_t i = 0; i < n_long; ++i) {
        const uint2 d = T.desc[T.d0 + S.ties[i]];
        const uint32_t len = long_len(d.x);
        for (uint32_t j = threadIdx.x; j < len && !*stop; j += NT) one(d.y, d.x + j);
    }
}

// One (gene, target) row with more columns than the table holds: its sums in direct-addressed
// blocks of column genes.
template <typename SH>
struct GtDense {
    static constexpr bool FILT = SH::kFilt;
    static constexpr uint32_t NT = SH::NT, kCols = SH::kWords / (FILT ? 3 : 1);  // columns per block (FILT: three arrays)
    const GtList &T;
    const CandFilter &cf;
    uint32_t *acc;
    GtLds<SH::NT> &S;
    uint32_t g, t, ncols, nr, nblk;
    const uint32_t *cw;

    __device__ __forceinline__ GtDense(uint32_t v, const GtList &T_, uint32_t n_tgt, const CandFilter &cf_, uint32_t *lds,
                                       GtLds<SH::NT> &S_)
        : T(T_), cf(cf_), acc(lds), S(S_) {
        g = v / n_tgt;
        t = v % n_tgt;
        ncols = S.tn[t];
        nr = S.nr[g];
        cw = S.tw[t];
        nblk = (ncols + kCols - 1) / kCols;
    }
    // The sums of columns c0 on; S.over stays zero.  Contains barriers.
    __device__ __forceinline__ void fill(uint32_t c0) {
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < (FILT ? 3 : 1) * kCols; i += NT) acc[i] = 0;
        if (threadIdx.x == 0) S.many = 0;
        __syncthreads();
        gt_walk<NT>(T, g, g + 1, S, [&](uint32_t, uint32_t rc, uint32_t x, uint32_t c, uint32_t pc) {
            if (S.tmap[x] != t || c - c0 >= kCols) return;
            atomicAdd(&acc[c - c0], min(rc, pc));
            if (FILT) {
                atomicAdd(&acc[kCols + c - c0], rc);
                atomicAdd(&acc[2 * kCols + c - c0], pc);
            }
        });
        __syncthreads();
    }
    // Sum of minima (0: no candidate) and of maxima of column c0 + i.
    __device__ __forceinline__ void value(uint32_t c0, uint32_t i, uint32_t *m, uint32_t *d) const {
        *m = c0 + i < ncols ? acc[i] : 0u;
        *d = 0;
        if (!*m) return;
        const uint32_t nc = load_global(cw + c0 + i);
        if (FILT && !candidate(cf, nr, nc, acc[kCols + i], acc[2 * kCols + i])) {
            *m = 0;
            return;
        }
        *d = nr + nc - *m;
    }
};

// Such a row, each block swept for the maximum, then for the ties.
template <typename SH>
__device__ void gt_dense_row(uint32_t v, const GtList &T, uint32_t n_tgt, uint32_t row0, const CandFilter &cf, uint32_t *lds,
                             GtLds<SH::NT> &S, uint32_t *__restrict__ bh_ptr, uint4 *__restrict__ slab, const GtCols &cmx) {
    using Dense = GtDense<SH>;
    constexpr uint32_t NT = SH::NT, kCols = Dense::kCols;
    Dense D(v, T, n_tgt, cf, lds, S);
    const uint32_t grow = S.trow[D.t] + row0 + D.g, col = S.tcol[D.t], nblk = D.nblk;
    if (threadIdx.x == 0) {
        S.best[v] = 0;
        S.cand_n = 0;
        S.over = 0;
    }
    for (uint32_t b = 0; b < nblk; ++b) {
        D.fill(b * kCols);
        for (uint32_t i = threadIdx.x; i < kCols; i += NT) {
            uint32_t m, d;
            D.value(b * kCols, i, &m, &d);
            if (!m) continue;
            if (col != UINT32_MAX && colmax_raise(cmx.key, col + b * kCols + i, m, d)) {
                const uint64_t idx = atomicAdd(cmx.count, 1ull);
                if (idx < cmx.cap) cmx.cands[idx] = make_uint4(col + b * kCols + i, row0 + D.g, m, d);
            }
            const unsigned long long want = (static_cast<unsigned long long>(m) << 32) | d;
            unsigned long long cur = S.best[v];
            for (;;) {
                const uint32_t om = static_cast<uint32_t>(cur >> 32), od = static_cast<uint32_t>(cur);
                if (om && !j_greater(m, d, om, od)) break;
                const unsigned long long prev = atomicCAS(&S.best[v], cur, want);
                if (prev == cur) break;
                cur = prev;
            }
        }
    }
    __syncthreads();
    const uint32_t bm = static_cast<uint32_t>(S.best[v] >> 32), bd = static_cast<uint32_t>(S.best[v]);
    if (bm) {
        for (uint32_t pass = 0; pass < 2; ++pass) {  // ties to the slab, or all of them to the candidates
            if (pass && S.cand_n <= kSlab) break;   // uniform: read after a barrier
            for (uint32_t b = 0; b < nblk; ++b) {
                if (nblk > 1) D.fill(b * kCols);  // a single block still holds its sums
                for (uint32_t i = threadIdx.x; i < kCols; i += NT) {
                    uint32_t m, d;
                    D.value(b * kCols, i, &m, &d);
                    if (!m || !j_equal(m, d, bm, bd)) continue;
                    if (!pass) {
                        const uint32_t n = atomicAdd(&S.cand_n, 1u);
                        if (n < kSlab) slab[static_cast<uint64_t>(grow) * kSlab + n] = make_uint4(b * kCols + i, m, d, 0);
                    } else {
                        const uint64_t idx = atomicAdd(cmx.count, 1ull);
                        if (idx < cmx.cap) cmx.cands[idx] = make_uint4(grow, b * kCols + i, m, d);
                    }
                }
            }
            __syncthreads();
        }
    }
    if (threadIdx.x == 0) {
        const uint32_t n = S.cand_n;
        if (n > kSlab) cmx.key[grow] = colmax_key(bm, bd);
        bh_ptr[grow] = n > kSlab ? 0u : n;
    }
    __syncthreads();
}

// Rows [v0, v1) summed in the hash table, their best values and tie counts cleared; false (uniform) when
// it is too small for them.
template <typename SH>
__device__ __forceinline__ bool gt_sum(uint32_t v0, uint32_t v1, const GtList &T, uint32_t n_tgt, uint32_t *lds,
                                       GtLds<SH::NT> &S) {
    constexpr bool FILT = SH::kFilt;
    constexpr uint32_t NT = SH::NT;
    uint32_t *hk = lds, *hv = lds + SH::kSlots, *hs = lds + 2 * SH::kSlots;
    const uint32_t tid = threadIdx.x;
    uint4 *z = reinterpret_cast<uint4 *>(lds);
    for (uint32_t i = tid; i < SH::kWords / 4; i += NT) z[i] = make_uint4(0, 0, 0, 0);
    if (tid == 0) {
        S.over = 0;
        S.cand_n = 0;
        S.many = 0;
    }
    __syncthreads();
    gt_walk<NT>(T, v0 / n_tgt, (v1 + n_tgt - 1) / n_tgt, S,
            [&](uint32_t g, uint32_t rc, uint32_t x, uint32_t c, uint32_t pc) {
        const uint32_t t = S.tmap[x];
        const uint32_t v = g * n_tgt + t;
        if (t == 255u || v - v0 >= v1 - v0) return;
        const uint32_t key = ((v << 24) | c) + 1u;  // genes stay below 2^24 - 1, so no wrap to 0
        uint32_t h = (key * 2654435761u) >> (32 - SH::kBits);
        for (uint32_t probe = 0;; ++probe) {  // a pair meets ~20 k-mers: mostly the key is there already
            uint32_t prev = *reinterpret_cast<volatile uint32_t *>(&hk[h]);
            if (prev == 0u) prev = atomicCAS(&hk[h], 0u, key);
            if (prev == 0u || prev == key) break;
            if (probe == kGtMaxProbe) {
                S.over = 1;
                return;
            }
            h = (h + 1) & (SH::kSlots - 1);
        }
        atomicAdd(&hv[h], min(rc, pc));
        if (FILT) atomicAdd(&hs[h], rc | (pc << 16));  // each half stays below 2^16: no carry
    });
    __syncthreads();
    const bool over = S.over != 0;
    for (uint32_t v = v0 + tid; v < v1; v += NT) {
        S.best[v] = 0;
        S.ties[v] = 0;
    }
    if (tid == 0) S.many = 0;
    __syncthreads();  // every thread has read the flag before the next call clears it
    return !over;
}

// Rows [v0, v1) through the hash table; false (uniform) when it is too small for them.
template <typename SH>
__device__ __forceinline__ bool gt_hashed(uint32_t v0, uint32_t v1, const GtList &T, uint32_t n_tgt,
                                          uint32_t row0, const CandFilter &cf, uint32_t *lds, GtLds<SH::NT> &S,
                                          uint32_t *__restrict__ bh_ptr, uint4 *__restrict__ slab, const GtCols &cmx) {
    constexpr bool FILT = SH::kFilt;
    constexpr uint32_t NT = SH::NT;
    uint32_t *hk = lds, *hv = lds + SH::kSlots, *hs = lds + 2 * SH::kSlots;
    const uint32_t tid = threadIdx.x;
    if (!gt_sum<SH>(v0, v1, T, n_tgt, lds, S)) return false;
    uint32_t ncw[SH::kPer], app = 0;
#pragma unroll
    for (uint32_t q = 0; q < SH::kPer; ++q) {  // the columns' window counts, gathered together
        const uint32_t key = hk[q * NT + tid];
        ncw[q] = 0;
        if (!key) continue;
        const uint32_t t = S.vt[(key - 1) >> 24], c = (key - 1) & 0xFFFFFFu;
        if (c < S.tn[t]) ncw[q] = load_global(S.tw[t] + c);
    }
#pragma unroll
    for (uint32_t q = 0; q < SH::kPer; ++q) {
        const uint32_t sl = q * NT + tid;
        const uint32_t key = hk[sl];
        if (!key) continue;
        const uint32_t v = (key - 1) >> 24, nr = S.nr[S.vr[v]], nc = ncw[q];
        uint32_t m = hv[sl];
        if (FILT && !candidate(cf, nr, nc, hs[sl] & 0xFFFFu, hs[sl] >> 16)) m = 0;
        if (!nc) m = 0;  // a gene that shares a k-mer has windows
        hv[sl] = m | (nc << 16);
        if (!m) continue;
        const uint32_t d = nr + nc - m, col = S.tcol[S.vt[v]];
        if (col != UINT32_MAX && colmax_raise(cmx.key, col + ((key - 1) & 0xFFFFFFu), m, d)) app |= 1u << q;
        const unsigned long long want = (static_cast<unsigned long long>(m) << 32) | d;
        unsigned long long cur = S.best[v];
        for (;;) {
            const uint32_t om = static_cast<uint32_t>(cur >> 32), od = static_cast<uint32_t>(cur);
            if (om && !j_greater(m, d, om, od)) break;
            const unsigned long long prev = atomicCAS(&S.best[v], cur, want);
            if (prev == cur) break;
            cur = prev;
        }
    }
    __syncthreads();
    // ties per row, the first kSlab of them to the row's slab
    uint32_t tie = 0;
#pragma unroll
    for (uint32_t q = 0; q < SH::kPer; ++q) {
        const uint32_t sl = q * NT + tid;
        const uint32_t key = hk[sl], m = hv[sl] & 0xFFFFu;
        if (!key || !m) continue;
        const uint32_t v = (key - 1) >> 24, g = S.vr[v], d = S.nr[g] + (hv[sl] >> 16) - m;
        const unsigned long long b = S.best[v];
        if (!j_equal(m, d, static_cast<uint32_t>(b >> 32), static_cast<uint32_t>(b))) continue;
        tie |= 1u << q;
        const uint32_t n = atomicAdd(&S.ties[v], 1u);
        if (n < kSlab)
            slab[static_cast<uint64_t>(S.trow[S.vt[v]] + row0 + g) * kSlab + n] = make_uint4((key - 1) & 0xFFFFFFu, m, d, 0);
    }
    __syncthreads();
    for (uint32_t v = v0 + tid; v < v1; v += NT) {
        const uint32_t n = S.ties[v], grow = S.trow[S.vt[v]] + row0 + S.vr[v];
        const unsigned long long b = S.best[v];
        if (n > kSlab) {  // every tie of the row becomes a candidate below
            S.many = 1;
            cmx.key[grow] = colmax_key(static_cast<uint32_t>(b >> 32), static_cast<uint32_t>(b));
        }
        bh_ptr[grow] = n > kSlab ? 0u : n;
    }
    __syncthreads();
    // candidates: pairs at their column's running maximum, and the ties of rows past the slab
    uint32_t big = 0;
    if (S.many)
#pragma unroll
        for (uint32_t q = 0; q < SH::kPer; ++q)
            if (((tie >> q) & 1u) && S.ties[(hk[q * NT + tid] - 1) >> 24] > kSlab) big |= 1u << q;
    const uint32_t mine = __popc(app) + __popc(big);
    uint32_t off = mine ? atomicAdd(&S.cand_n, mine) : 0u;
    __syncthreads();
    if (tid == 0 && S.cand_n) S.cand_base = atomicAdd(cmx.count, static_cast<unsigned long long>(S.cand_n));
    __syncthreads();
    if (mine) {
#pragma unroll
        for (uint32_t q = 0; q < SH::kPer; ++q) {
            if (!(((app | big) >> q) & 1u)) continue;
            const uint32_t sl = q * NT + tid;
            const uint32_t key = hk[sl], c = (key - 1) & 0xFFFFFFu, v = (key - 1) >> 24, m = hv[sl] & 0xFFFFu;
            const uint32_t g = S.vr[v], t = S.vt[v], d = S.nr[g] + (hv[sl] >> 16) - m;
            if ((app >> q) & 1u) {
                const uint64_t idx = S.cand_base + off++;
                if (idx < cmx.cap) cmx.cands[idx] = make_uint4(S.tcol[t] + c, row0 + g, m, d);
            }
            if ((big >> q) & 1u) {
                const uint64_t idx = S.cand_base + off++;
                if (idx < cmx.cap) cmx.cands[idx] = make_uint4(S.trow[t] + row0 + g, c, m, d);
            }
        }
    }
    __syncthreads();  // the table takes the next rows
    return true;
}

// What both tile kernels read.
struct GtArgs {
    const DevGroupDict *__restrict__ dicts;
    const DevGroupTgt *__restrict__ tgts;
    const uint8_t *__restrict__ tmap;
    const DevGroupTile *__restrict__ tiles;
    const uint32_t *__restrict__ cursor;
    const uint2 *__restrict__ desc;
    const uint32_t *__restrict__ post;
    const uint32_t *__restrict__ aux;
    uint32_t gene_bits;
    CandFilter cf;
    uint32_t *__restrict__ bh_ptr;
    uint4 *__restrict__ slab;
    GtCols cmx;
    uint2 *__restrict__ big;       // tiles left to the big kernel: (tile, first row)
    uint32_t *__restrict__ n_big;
};

// A tile: its descriptors, rows ((gene, target) pairs), targets per gene, first gene.
struct GtTile {
    GtList T;
    uint32_t rows, n_tgt, g0;
    CandFilter cf;
};
// Ends with a barrier.
template <uint32_t NT>
__device__ __forceinline__ GtTile gt_open(const GtArgs &A, uint32_t tile, GtLds<NT> &S) {
    const uint32_t tid = threadIdx.x;
    const DevGroupTile tl = A.tiles[tile];
    const DevGroupDict &d = A.dicts[tl.dict];
    GtTile R{GtList{A.desc, A.post, A.aux, A.gene_bits, 0, 0, 0, 0}, tl.ng * d.n_tgt, d.n_tgt, tl.g0, A.cf};
    R.cf.k = d.k;
    for (uint32_t t = tid; t < R.n_tgt; t += NT) {
        const DevGroupTgt g = A.tgts[d.tgt_base + t];
        S.tw[t] = g.nwin;
        S.tn[t] = g.n_genes;
        S.trow[t] = g.row_base;
        S.tcol[t] = g.col_base;
    }
    for (uint32_t x = tid; x < d.n_dicts; x += NT) S.tmap[x] = A.tmap[d.tmap_base + x];
    for (uint32_t g = tid; g < tl.ng; g += NT) S.nr[g] = load_global(d.nwin + tl.g0 + g);
    for (uint32_t r = tid; r < R.rows; r += NT) {
        S.vr[r] = static_cast<uint8_t>(r / R.n_tgt);
        S.vt[r] = static_cast<uint8_t>(r % R.n_tgt);
    }
    R.T.d0 = d.desc_base + load_global(d.mv_ptr + tl.g0);
    R.T.nd = A.cursor[static_cast<uint64_t>(tile) * kGroupCursorStride] - R.T.d0;
    R.T.i0 = A.cursor[static_cast<uint64_t>(tile) * kGroupCursorStride + 1];
    R.T.ni = d.desc_base + load_global(d.mv_ptr + tl.g0 + tl.ng) - R.T.i0;
    __syncthreads();
    return R;
}

// One tile from its row v on.  The small shape gives up on a tile whose rows do not fit its table after one
// halving and lists what is left.
template <typename SH, bool LAST>
__device__ __forceinline__ void gt_tile(const GtArgs &A, uint32_t tile, uint32_t v, uint32_t *lds, GtLds<SH::NT> &S) {
    const uint32_t tid = threadIdx.x;
    const GtTile R = gt_open<SH::NT>(A, tile, S);
    if (R.T.nd + R.T.ni == 0) {  // the genes share no k-mer with any target
        for (uint32_t r = tid; r < R.rows; r += SH::NT) A.bh_ptr[S.trow[S.vt[r]] + R.g0 + S.vr[r]] = 0;
        return;
    }
    uint32_t step = R.rows;
    while (v < R.rows) {
        const uint32_t v1 = min(R.rows, v + step);
        if (gt_hashed<SH>(v, v1, R.T, R.n_tgt, R.g0, R.cf, lds, S, A.bh_ptr, A.slab, A.cmx)) {
            v = v1;
            if (LAST) step = min(2 * step, R.rows);  // a gene of many columns holds up its own rows only
        } else if (!LAST && step < R.rows) {
            if (tid == 0) A.big[atomicAdd(A.n_big, 1u)] = make_uint2(tile, v);
            return;
        } else if (v1 - v > 1) {
            step = (v1 - v + 1) / 2;
        } else {
            gt_dense_row<SH>(v, R.T, R.n_tgt, R.g0, R.cf, lds, S, A.bh_ptr, A.slab, A.cmx);
            ++v;
        }
    }
}

// Calls f(row, column, m, d) for every pair of a tile whose value is the final maximum of its column's
// best-hit row (column maxima) or of its own row (rows with ties past the slab, whose key is set).
template <typename SH, typename F>
__device__ __forceinline__ void gt_replay(const GtArgs &A, uint32_t tile, uint32_t *lds, GtLds<SH::NT> &S, F f) {
    using Dense = GtDense<SH>;
    const GtTile R = gt_open<SH::NT>(A, tile, S);
    if (R.T.nd + R.T.ni == 0) return;
    auto pair = [&](uint32_t g, uint32_t t, uint32_t c, uint32_t m, uint32_t d) {
        const unsigned long long key = colmax_key(m, d);
        const uint32_t grow = S.trow[t] + R.g0 + g;
        if (A.cmx.key[grow] == key) f(grow, c, m, d);
        if (S.tcol[t] != UINT32_MAX && A.cmx.key[S.tcol[t] + c] == key) f(S.tcol[t] + c, R.g0 + g, m, d);
    };
    uint32_t step = R.rows;
    for (uint32_t v = 0; v < R.rows;) {
        const uint32_t v1 = min(R.rows, v + step);
        if (gt_sum<SH>(v, v1, R.T, R.n_tgt, lds, S)) {
            const uint32_t *hk = lds, *hv = lds + SH::kSlots, *hs = lds + 2 * SH::kSlots;
            for (uint32_t sl = threadIdx.x; sl < SH::kSlots; sl += SH::NT) {
                const uint32_t key = hk[sl];
                if (!key) continue;
                const uint32_t r = (key - 1) >> 24, c = (key - 1) & 0xFFFFFFu, g = S.vr[r], t = S.vt[r], nr = S.nr[g], m = hv[sl];
                const uint32_t nc = c < S.tn[t] ? load_global(S.tw[t] + c) : 0u;
                if (SH::kFilt && !candidate(R.cf, nr, nc, hs[sl] & 0xFFFFu, hs[sl] >> 16)) continue;
                if (m && nc) pair(g, t, c, m, nr + nc - m);
            }
            v = v1;
            step = min(2 * step, R.rows);
        } else if (v1 - v > 1) {
            step = (v1 - v + 1) / 2;
        } else {
            Dense D(v, R.T, R.n_tgt, R.cf, lds, S);
            if (threadIdx.x == 0) S.over = 0;
            for (uint32_t b = 0; b < D.nblk; ++b) {
                D.fill(b * Dense::kCols);
                for (uint32_t i = threadIdx.x; i < Dense::kCols; i += SH::NT) {
                    uint32_t m, d;
                    D.value(b * Dense::kCols, i, &m, &d);
                    if (m) pair(D.g, D.t, b * Dense::kCols + i, m, d);
                }
            }
            ++v;
        }
        __syncthreads();  // the table takes the next rows
    }
}

// One tile.  50 genomes of 3000 to 5000 genes: 0.71 ms, of which the walk takes 0.38 (random runs of
// postings; 1.15 ms in all with eight lanes per descriptor and 8-byte postings), the table's keys 0.07, sums,
// values and ties 0.08, and the column keys' device atomics with the candidates 0.18 (timed by leaving each
// out).  Bound by latency: its waves wait 77% of their cycles, VALU issues in 36% and LDS is busy in 23% of
// the kernel's; 26 KiB of LDS, six work-groups per CU.
template <bool FILT>
__global__ __launch_bounds__(kGtThreads) void k_group_tile(GtArgs A) {
    using SH = GtSmall<FILT>;
    __shared__ __align__(16) uint32_t lds[SH::kWords];
    __shared__ GtLds<SH::NT> S;
    gt_tile<SH, false>(A, xcd_item(blockIdx.x, gridDim.x), 0, lds, S);
}

// The tiles with more columns than that (genes with a k-mer that many genes share; letters used unevenly),
// in a table of eight times the sums (FILT: four).
template <bool FILT>
__global__ __launch_bounds__(kGtThreadsBig) void k_group_tile_big(GtArgs A) {
    using SH = GtBig<FILT>;
    extern __shared__ __align__(16) uint32_t gt_dyn[];
    __shared__ GtLds<SH::NT> S;
    const uint32_t n = *A.n_big;
    for (uint32_t i = blockIdx.x; i < n; i += gridDim.x) {  // uniform
        const uint2 job = A.big[i];
        gt_tile<SH, true>(A, job.x, job.y, gt_dyn, S);
        __syncthreads();
    }
}

// Hits from the group tiles' candidates, as k_colmax_rows: every listed pair still at its row's final
// maximum.  How many pairs are listed on the way there depends on the order of the tiles; when there were
// more than the list holds, the tiles are replayed with the final maxima instead, which lists nothing.  The
// number of hits is then what the caller's capacity has to hold (it is below the list's otherwise): a plan
// fails on the same inputs every time or never, and needed is exact.
template <bool FILT>
__global__ __launch_bounds__(kGtThreads) void k_group_rows(GtArgs A, uint32_t n_tiles, ColRows R, unsigned long long *n_hits,
                                                           uint64_t hit_cap, pdp_status *st) {
    using SH = GtSmall<FILT>;
    const uint64_t n = *A.cmx.count;
    if (n <= A.cmx.cap) {
        for (uint64_t i = blockIdx.x * uint64_t(kGtThreads) + threadIdx.x; i < n; i += gridDim.x * uint64_t(kGtThreads)) {
            const uint4 c = A.cmx.cands[i];
            if (colmax_key(c.z, c.w) == A.cmx.key[c.x]) colmax_count(R, c.x, c.y, c.z, c.w);
        }
        return;
    }
    __shared__ __align__(16) uint32_t lds[SH::kWords];
    __shared__ GtLds<SH::NT> S;
    uint32_t hits = 0;
    for (uint32_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        gt_replay<SH>(A, tile, lds, S, [&](uint32_t row, uint32_t col, uint32_t m, uint32_t d) {
            colmax_count(R, row, col, m, d);
            ++hits;
        });
        __syncthreads();
    }
    hits = wave_sum(hits);
    if (lane_id() == 0 && hits) {
        const unsigned long long so_far = atomicAdd(n_hits, static_cast<unsigned long long>(hits)) + hits;
        if (so_far > hit_cap) raise_status(st, PDP_E_CAPACITY, so_far, 0);  // the last one's is the total
    }
}

// After the row pointers, as k_colmax_big: hits of rows with more than kSlab of them.
template <bool FILT>
__global__ __launch_bounds__(kGtThreads) void k_group_big(GtArgs A, uint32_t n_tiles, const uint32_t *__restrict__ n_big,
                                                          ColCsr C) {
    using SH = GtSmall<FILT>;
    if (*n_big == 0u) return;
    const uint64_t n = *A.cmx.count;
    if (n <= A.cmx.cap) {
        for (uint64_t i = blockIdx.x * uint64_t(kGtThreads) + threadIdx.x; i < n; i += gridDim.x * uint64_t(kGtThreads)) {
            const uint4 c = A.cmx.cands[i];
            if (colmax_key(c.z, c.w) == A.cmx.key[c.x]) colmax_write(C, c.x, c.y, c.z, c.w);
        }
        return;
    }
    __shared__ __align__(16) uint32_t lds[SH::kWords];
    __shared__ GtLds<SH::NT> S;
    for (uint32_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        gt_replay<SH>(A, tile, lds, S,
                      [&](uint32_t row, uint32_t col, uint32_t m, uint32_t d) { colmax_write(C, row, col, m, d); });
        __syncthreads();
    }
}

// ------------------------------------------------------------------ host

hipError_t launch_group_join(const PlanShape &p, const PairWs &w, hipStream_t s) {
    if (!p.n_gdicts) return hipSuccess;
    const uint32_t dyn = sizeof(GjDict) * p.gmax_dicts;
    const GjOut out{w.gpost, w.gaux, w.gdesc, w.gcursor, p.gene_bits};
    if (p.n_gitems) {
        hipLaunchKernelGGL(k_group_join<false>, dim3(p.n_gitems), dim3(kGjThreads), dyn, s, w.gdicts, w.gitems, w.gbig,
                           w.n_gbig, out);
        PDP_TRY(hipGetLastError());
        hipLaunchKernelGGL(k_group_join_big<false>, dim3(std::min(p.n_gitems, kGjBigGrid)), dim3(kGjThreads), dyn, s, w.gdicts,
                           w.gitems, w.gbig, w.n_gbig, out);
        PDP_TRY(hipGetLastError());
    }
    if (p.n_gitems_wide) {
        const DevGroupItem *items = w.gitems + p.n_gitems;
        uint2 *big = w.gbig + p.n_gitems + group_pieces(p);
        uint32_t *n_big = w.n_gbig + 1;
        hipLaunchKernelGGL(k_group_join<true>, dim3(p.n_gitems_wide), dim3(kGjThreads), dyn, s, w.gdicts, items, big, n_big,
                           out);
        PDP_TRY(hipGetLastError());
        hipLaunchKernelGGL(k_group_join_big<true>, dim3(std::min(p.n_gitems_wide, kGjBigGrid)), dim3(kGjThreads), dyn, s,
                           w.gdicts, items, big, n_big, out);
        PDP_TRY(hipGetLastError());
    }
    return hipSuccess;
}

hipError_t allow_group_lds() {
    for (const void *f : {reinterpret_cast<const void *>(k_group_tile_big<false>), reinterpret_cast<const void *>(k_group_tile_big<true>)})
        PDP_TRY(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 4 * GtBig<false>::kWords));
    return hipSuccess;
}

template <bool FILT>
static hipError_t group_tiles(const PlanShape &p, const GtArgs &A, hipStream_t s) {
    hipLaunchKernelGGL(k_group_tile<FILT>, dim3(p.n_gtiles), dim3(kGtThreads), 0, s, A);
    PDP_TRY(hipGetLastError());
    hipLaunchKernelGGL(k_group_tile_big<FILT>, dim3(std::min(p.n_gtiles, kGtBigGrid)), dim3(kGtThreadsBig),
                       4 * GtBig<FILT>::kWords, s, A);
    return hipGetLastError();
}

static GtArgs group_args(const PlanShape &p, const PairWs &w, pdp_bh_out *bh) {
    const GtCols cmx{w.colkey, w.cands + p.cand_cap, w.gcand_count, p.gcand_cap};
    const CandFilter cf{0, p.theta_n, p.theta_d, p.tau_n, p.tau_d};
    return GtArgs{w.gdicts, w.gtgts, w.tmap, w.gtiles, w.gcursor, w.gdesc, w.gpost, w.gaux, p.gene_bits, cf, bh->ptr, w.slab, cmx,
                  w.gbig_tiles, w.n_gbig + 2};
}

hipError_t launch_group_tiles(const PlanShape &p, const PairWs &w, pdp_bh_out *bh, hipStream_t s) {
    if (!p.n_gtiles) return hipSuccess;
    const GtArgs A = group_args(p, w, bh);
    return p.theta_d || p.tau_d ? group_tiles<true>(p, A, s) : group_tiles<false>(p, A, s);
}

static dim3 group_rows_grid(const PlanShape &p) {
    return dim3(static_cast<uint32_t>(std::max<uint64_t>(1, std::min<uint64_t>(2048, (p.gcand_cap + kGtThreads - 1) / kGtThreads))));
}

hipError_t launch_group_rows(const PlanShape &p, const PairWs &w, pdp_bh_out *bh, pdp_status *st, hipStream_t s) {
    if (!p.n_gtiles) return hipSuccess;
    const GtArgs A = group_args(p, w, bh);
    const ColRows R{bh->ptr, w.slab, w.colcursor, w.big_rows, w.n_big};
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, group_rows_grid(p), dim3(kGtThreads), 0, s, A, p.n_gtiles, R, w.n_ghits, p.ghit_cap, st);
    };
    if (p.theta_d || p.tau_d) launch(k_group_rows<true>);
    else launch(k_group_rows<false>);
    return hipGetLastError();
}

hipError_t launch_group_big(const PlanShape &p, const PairWs &w, pdp_bh_out *bh, hipStream_t s) {
    if (!p.n_gtiles) return hipSuccess;
    const GtArgs A = group_args(p, w, bh);
    const ColCsr C{bh->ptr, bh->col, bh->num, bh->den, bh->capacity, w.colcursor};
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, group_rows_grid(p), dim3(kGtThreads), 0, s, A, p.n_gtiles, w.n_big, C);
    };
    if (p.theta_d || p.tau_d) launch(k_group_big<true>);
    else launch(k_group_big<false>);
    return hipGetLastError();
}

}  // namespace pdp
