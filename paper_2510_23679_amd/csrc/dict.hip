// k-mer dictionary build for one or many genomes on gfx950, in one set of launches.
//
// 1. k_mv_wave: one wave per gene encodes every window g[p..p+k-1] into a
//    code of 5 bits per amino acid or 2 per nucleotide (a lane's windows are
//    consecutive, so each code is the previous one shifted by one letter),
//    sorts the codes in registers (a bitonic network of
//    kMvWaveCap keys, eight per lane, lanes exchanging by shuffles) and
//    run-length encodes them into the gene's multiplicity vector (Multiplicity
//    vector building phase, Alg. 1: group equal identifiers, count, ascending
//    order).  Longer genes are queued by size for k_mv_mid and k_mv_rest (one work-group
//    per gene, 8, 16 or 32 codes per thread sorted in registers, exchanges
//    across waves through LDS; past kMvSortCap windows codes sorted in
//    global memory).
// 2. A scan of the distinct-k-mer counts of all genes gives the CSR offsets,
//    and k_mv_compact packs the vectors (and notes each entry's gene).
// 3. The inverted index (all entries ordered by k-mer code, ties by gene) is a
//    two-level partition: the leading-letter buckets are grouped into coarse
//    bins of 2^s buckets (s per genome, up to kIxBinTarget entries per bin); k_ix_hist
//    counts bins per block of entries in LDS and adds them to the bin totals
//    (one global atomic per block and bin), a scan gives every bin its output
//    range, k_ix_place hands each block a run of every bin's range (again one
//    atomic per block and bin) and drops its entries there by LDS rank, and
//    k_ix_sort_bin sorts each bin by (code, gene) in LDS (a counting sort by
//    bucket and the next one or two letters, which leaves about one entry per
//    slot, then ranks inside each slot) and writes the bin's part of the
//    bucket directory.
// Genes and buckets of all genomes of a call are numbered consecutively; a
// work-group finds its genome by binary search over the per-genome bases.
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "internal.hpp"

namespace pdp {

constexpr uint32_t kMvThreads = 256;
static_assert(kMvSortCap == kMvThreads * 32, "the largest k_mv_mid class sorts 32 codes per thread");
constexpr uint32_t kIxBatch = 8;  // index entries a thread loads per round in the histogram and placement
constexpr uint32_t kDescPerLaunch = 16;
constexpr uint32_t kBuildCounters = 8;  // [0..3] genes queued per size class, [4] ended histogram blocks

struct DescChunk {
    uint32_t first, count;
    DevBuild d[kDescPerLaunch];
};
static_assert(sizeof(DescChunk) <= 4096, "descriptor chunks travel as kernel arguments");

// Set-up of a build: descriptors passed by value into the workspace table (kernel arguments are
// captured at launch, so the host copy may go away at once), their genomes' statuses cleared and
// the CSR of a genome without genes written (nothing else writes it).  The first chunk's launch also
// zeroes the build's counters and the bin totals (total_bins of them).
__global__ __launch_bounds__(256) void k_build_init(DevBuild *table, DescChunk c, uint32_t *counters, uint32_t *bintot,
                                                    uint32_t total_bins) {
    const uint32_t i0 = blockIdx.x * 256 + threadIdx.x, stride = gridDim.x * 256;
    if (i0 < c.count) {
        const DevBuild &d = c.d[i0];
        table[c.first + i0] = d;
        d.status->code = 0;
        d.status->flags = 0;
        d.status->needed = 0;
        d.status->where = ~0ull;
        if (d.n_genes == 0) d.mv_ptr[0] = 0;
    }
    if (c.first) return;
    if (i0 < kBuildCounters) counters[i0] = 0;
    for (uint32_t b = i0; b < total_bins; b += stride) bintot[b] = 0;
}

__device__ __forceinline__ uint32_t find_genome_by_gene(const DevBuild *t, uint32_t n, uint32_t gene) {
    uint32_t lo = 0, hi = n - 1;
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) >> 1;
        if (t[mid].gene_base <= gene) lo = mid;
        else hi = mid - 1;
    }
    // genomes without genes share a base with the next one; take the last with genes
    return lo;
}


// Orders LDS writes of a wave before its later LDS reads (a wave runs in lock step,
// so no work-group barrier is needed).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The value of x in lane (this lane ^ lj), lj a power of two below kWave, without an LDS
// round trip where the lane pattern allows: DPP moves for 1 and 2 (quad permutations) and 8
// (rotation by 8 inside each row of 16 lanes), ds_swizzle in bit-mask mode (lanes of a half
// wave, no address operand) for 4 and 16, ds_bpermute for 32.  Every lane of the wave must
// be active.
__device__ __forceinline__ uint32_t xor_lanes32(uint32_t x, uint32_t lj) {
    const int v = static_cast<int>(x);
    switch (lj) {
        case 1: return static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true));
        case 2: return static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true));
        case 8: return static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(v, 0x128, 0xF, 0xF, true));
        case 4: return static_cast<uint32_t>(__builtin_amdgcn_ds_swizzle(v, 0x101F));
        case 16: return static_cast<uint32_t>(__builtin_amdgcn_ds_swizzle(v, 0x401F));
        default: return __shfl_xor(x, lj, kWave);
    }
}
// The middle of three values (v_med3_u32): with bound 0 the smaller of a and b, with all ones the
// larger, so a comparator whose direction depends on the lane takes one instruction per output.
__device__ __forceinline__ uint32_t pick(uint32_t a, uint32_t b, uint32_t bound) {
    uint32_t r;
    asm("v_med3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(bound));  // asm: the compiler does not end on a network of the min / max form
    return r;
}
// All ones in lanes with bit b of the lane number set.
__device__ __forceinline__ uint32_t lane_bit_mask(uint32_t b) {
    return static_cast<uint32_t>(static_cast<int32_t>(lane_id() << (31u - b)) >> 31);
}
constexpr uint32_t log2_of(uint32_t x) { return x <= 1 ? 0 : 1 + log2_of(x >> 1); }

// The same network as below for 32-bit keys.  A comparator keeps the minimum where the lane bits of
// its distance and of its direction agree: their masks' exclusive or is the bound that picks it.
// 45 stages of 512 keys: 66 instructions a key where compare, select and exchange took ~115.
template <uint32_t E>
__device__ __forceinline__ void wave_bitonic_sort(uint32_t (&key)[E]) {
    constexpr uint32_t N = kWave * E;
    uint32_t bit[6];
#pragma unroll
    for (uint32_t b = 0; b < 6; ++b) bit[b] = lane_bit_mask(b);
#pragma unroll
    for (uint32_t size = 2; size <= N; size <<= 1) {
        // all ones in lanes that sort this run downwards (the last run goes up everywhere)
        const uint32_t down = size < E || size == N ? 0u : bit[log2_of(size / E)];
#pragma unroll
        for (uint32_t j = size >> 1; j > 0; j >>= 1) {
            if (j < E) {
#pragma unroll
                for (uint32_t e = 0; e < E; ++e) {
                    if (e & j) continue;
                    const uint32_t a = key[e], b = key[e | j];
                    if (size < E && (e & size)) {
                        key[e] = max(a, b);
                        key[e | j] = min(a, b);
                    } else if (size < E || size == N) {
                        key[e] = min(a, b);
                        key[e | j] = max(a, b);
                    } else {
                        key[e] = pick(a, b, down);
                        key[e | j] = pick(a, b, ~down);
                    }
                }
            } else {
                const uint32_t lj = j / E;
                const uint32_t bound = bit[log2_of(lj)] ^ down;
#pragma unroll
                for (uint32_t e = 0; e < E; ++e) key[e] = pick(key[e], xor_lanes32(key[e], lj), bound);
            }
        }
    }
}

// Ascending bitonic sort of kWave * E keys, E per lane in blocked order (lane l holds
// elements l*E .. l*E+E-1): comparators inside a lane swap registers, the others pair
// lanes by a shuffle and keep the minimum or maximum.
template <uint32_t E, typename K>
__device__ __forceinline__ void wave_bitonic_sort(K (&key)[E]) {
    constexpr uint32_t N = kWave * E;
    const uint32_t l = lane_id();
#pragma unroll
    for (uint32_t size = 2; size <= N; size <<= 1) {
#pragma unroll
        for (uint32_t j = size >> 1; j > 0; j >>= 1) {
            if (j < E) {
#pragma unroll
                for (uint32_t e = 0; e < E; ++e) {
                    if (e & j) continue;
                    const bool asc = ((l * E + e) & size) == 0;
                    const K a = key[e], b = key[e | j];
                    const bool sw = asc ? a > b : a < b;
                    key[e] = sw ? b : a;
                    key[e | j] = sw ? a : b;
                }
            } else {
                const uint32_t lj = j / E;
                const bool lower = (l & lj) == 0;
#pragma unroll
                for (uint32_t e = 0; e < E; ++e) {
                    const K o = __shfl_xor(key[e], lj, kWave);
                    const bool keep_min = lower == (((l * E + e) & size) == 0);
                    const K mn = o < key[e] ? o : key[e], mx = o < key[e] ? key[e] : o;
                    key[e] = keep_min ? mn : mx;
                }
            }
        }
    }
}

// Checks a gene's offsets and window count; on failure records the status and an empty
// vector and returns false.
__device__ __forceinline__ bool gene_ok(const DevBuild &B, uint32_t g, uint32_t G, uint32_t *dcnt, uint64_t *o,
                                        uint64_t *len, uint32_t *nw) {
    *o = B.off[g];
    const uint64_t e = B.off[g + 1];
    if (e < *o || e > B.n_residues) {
        if (lane_id() == 0) {
            raise_status(B.status, PDP_E_INVAL, 0, g);
            B.nwin[g] = 0;
            dcnt[G] = 0;
        }
        return false;
    }
    *len = e - *o;
    const uint64_t nw64 = *len >= B.k ? *len - B.k + 1 : 0;
    if (nw64 > B.max_windows) {
        if (lane_id() == 0) {
            raise_status(B.status, PDP_E_LIMIT, nw64, g);
            B.nwin[g] = 0;
            dcnt[G] = 0;
        }
        return false;
    }
    *nw = static_cast<uint32_t>(nw64);
    return true;
}

// Amino-acid k-mers of 7 letters take 35 bits as 5-bit codes but only 31 as base-20 values
// (20^7 < 2^31), and both order k-mers alike (letter by letter, first letter most
// significant).  For such genomes the multiplicity-vector sorts run on 32-bit base-20 keys, and
// each distinct key is turned back into its 5-bit code when the vector is written.
__device__ __forceinline__ bool base20_keys(const DevBuild &B) { return B.bits == 5u && B.k == 7u; }
constexpr uint32_t kPow20_6 = 64000000u;  // 20^(7-1): the weight of a 7-mer's first letter

__device__ __forceinline__ uint64_t base20_to_code(uint32_t v, uint32_t k) {
    uint64_t c = 0;
    for (uint32_t i = 0; i < k; ++i) {  // digits from the last letter on
        const uint32_t q = v / 20u;
        c |= static_cast<uint64_t>(v - q * 20u) << (5u * i);
        v = q;
    }
    return c;
}

// The keys of windows p0 .. p0+E-1 (those below nw; the rest sort last) from the gene's symbols:
// 5-bit codes, or base-20 values when B20; each window's key is the previous one shifted by one
// letter, so the first k-1 letters are read once.
template <uint32_t E, typename K, bool B20>
__device__ __forceinline__ void window_keys(const uint8_t *sym, uint32_t p0, uint32_t nw, uint32_t k, uint32_t bits,
                                            K (&key)[E]) {
    if constexpr (B20) {
        uint32_t c = 0;  // base-20 value of the k-1 letters after the window's first
        if (p0 < nw)
            for (uint32_t j = 0; j + 1 < k; ++j) c = c * 20u + sym[p0 + j];
#pragma unroll
        for (uint32_t e = 0; e < E; ++e) {
            const uint32_t p = p0 + e;
            uint32_t full = ~0u;
            if (p < nw) {
                full = c * 20u + sym[p + k - 1];
                c = full - sym[p] * kPow20_6;
            }
            key[e] = static_cast<K>(full);
        }
    } else {
        const uint64_t mask = (1ull << (bits * k)) - 1ull;  // bits * k <= 62
        uint64_t c = 0;
        if (p0 < nw)
            for (uint32_t j = 0; j + 1 < k; ++j) c = (c << bits) | sym[p0 + j];
#pragma unroll
        for (uint32_t e = 0; e < E; ++e) {
            const uint32_t p = p0 + e;
            if (p < nw) c = ((c << bits) | sym[p + k - 1]) & mask;
            key[e] = p < nw ? static_cast<K>(c) : static_cast<K>(~0ull);  // past the windows: sorts last
        }
    }
}

template <bool B20, typename K>
__device__ __forceinline__ uint64_t key_code(K key, uint32_t k) {
    if constexpr (B20) return base20_to_code(static_cast<uint32_t>(key), k);
    else return static_cast<uint64_t>(key);
}

constexpr uint32_t kMvWaveEMax = 16;
constexpr uint32_t kMvWaveCap = kWave * kMvWaveEMax;  // windows a wave sorts in registers
constexpr uint32_t kMvWaves = kMvThreads / kWave;

constexpr uint32_t kMvHalf = 512;  // sorted keys a wave passes through LDS at a time

// A key of the narrow form (32 bits: base-20 value or code) from a code, and back.
__device__ __forceinline__ uint32_t code_to_base20(uint64_t c, uint32_t k) {
    uint32_t v = 0;
    for (uint32_t i = 0; i < k; ++i) v = v * 20u + static_cast<uint32_t>((c >> (5u * (k - 1u - i))) & 31u);
    return v;
}
__device__ __forceinline__ uint32_t code_to_key(const DevBuild &B, uint64_t c) {
    return base20_keys(B) ? code_to_base20(c, B.k) : static_cast<uint32_t>(c);
}
__device__ __forceinline__ uint64_t key_to_code(const DevBuild &B, uint32_t key) {
    return base20_keys(B) ? base20_to_code(key, B.k) : key;
}

// One gene's multiplicity vector by one wave: codes E per lane in registers, sorted by the
// wave's bitonic network (E = 4, 8 or 16: the smallest that holds the gene).  The sorted keys then
// pass through LDS (kMvHalf at a time) so that consecutive lanes hold consecutive keys: run heads
// are ranked by ballots and the keys and counts go out in whole cache lines (each lane storing its
// own run of the blocked order touches 64 lines per store).  buf: kMvHalf keys over the gene's
// symbols; hp: kWave*E+1 head positions.
// K: the key type, 32 bits when the codes fit (bits * k <= 32), halving the shuffles.
// B20: base-20 keys (base20_keys).  NARROW: the slots take 32-bit keys instead of codes.
template <uint32_t E, typename K, bool B20, bool NARROW>
__device__ __forceinline__ void mv_wave_gene(const DevBuild &B, uint8_t *sym, uint16_t *hp, uint64_t o, uint32_t nw,
                                             uint32_t *cnt_out) {
    const uint32_t lane = lane_id();
    const uint32_t k = B.k;
    K key[E];
    // the lane's windows p0 .. p0+E-1 are consecutive
    window_keys<E, K, B20>(sym, lane * E, nw, k, B.bits, key);
    if constexpr (sizeof(K) == 4) wave_bitonic_sort<E>(key);
    else wave_bitonic_sort<E, K>(key);
    constexpr uint32_t kRounds = kWave * E > kMvHalf ? kWave * E / kMvHalf : 1;
    constexpr uint32_t kLanes = kWave / kRounds;  // lanes whose keys make one round
    K *buf = reinterpret_cast<K *>(sym);
    uint32_t total = 0;
    K last = 0;
#pragma unroll
    for (uint32_t h = 0; h < kRounds; ++h) {
        if (h * kMvHalf >= nw) break;  // uniform
        wave_lds_sync();
        if (lane / kLanes == h) {
#pragma unroll
            for (uint32_t e = 0; e < E; ++e) buf[(lane % kLanes) * E + e] = key[e];
        }
        wave_lds_sync();
#pragma unroll
        for (uint32_t q = 0; q < kLanes * E / kWave; ++q) {
            const uint32_t x = q * kWave + lane, i = h * kMvHalf + x;
            const K c = buf[x], prev = x ? buf[x - 1] : last;
            const bool head = i < nw && (i == 0 || c != prev);
            const uint64_t mask = __ballot(head);
            const uint32_t r = total + mask_below(mask);
            if (head) {
                hp[r] = static_cast<uint16_t>(i);
                if constexpr (NARROW) store_global(reinterpret_cast<uint32_t *>(B.slot_code) + o + r, static_cast<uint32_t>(c));
                else store_global(B.slot_code + o + r, key_code<B20>(c, k));
            }
            total += static_cast<uint32_t>(__popcll(mask));
        }
        last = buf[kLanes * E - 1];
    }
    if (lane == 0) hp[total] = static_cast<uint16_t>(nw);
    wave_lds_sync();
    for (uint32_t r = lane; r < total; r += kWave)
        store_global(B.slot_cnt + o + r, static_cast<uint32_t>(hp[r + 1]) - hp[r]);
    *cnt_out = total;
}

// Longer genes go to lists by size: counters[0] / long_list past kMvSortCap windows,
// counters[c] / mid_list + (c - 1) * stride for genes sorted 8 << (c - 1) codes a thread, c = 1, 2, 3.
// NARROW: every genome of the build sorts 32-bit keys (5-bit codes of at most 32 bits, or
// base-20 values): a separate instance without the 64-bit path, which needs fewer registers.
template <bool NARROW>
__global__ __launch_bounds__(kMvThreads) void k_mv_wave(const DevBuild *__restrict__ table, uint32_t n_genomes,
                                                        uint32_t total_genes, uint32_t *__restrict__ dcnt,
                                                        uint64_t *__restrict__ mid_list, uint64_t *__restrict__ long_list,
                                                        uint32_t stride, uint32_t *__restrict__ counters) {
    // symbols, then sorted keys
    constexpr uint32_t kBuf = (kMvHalf * (NARROW ? 4 : 8) + 15) / 16 * 16;
    static_assert(kBuf >= kMvWaveCap + kKMaxAll, "a gene's symbols fit");
    __shared__ __align__(16) uint8_t sym_all[kMvWaves][kBuf];
    __shared__ uint16_t hp_all[kMvWaves][kMvWaveCap + 1];
    const uint32_t w = threadIdx.x / kWave, lane = lane_id();
    const uint32_t G = blockIdx.x * kMvWaves + w;
    if (G >= total_genes) return;
    const uint32_t t = find_genome_by_gene(table, n_genomes, G);
    const DevBuild &B = table[t];
    const uint32_t g = G - B.gene_base;
    uint64_t o, len;
    uint32_t nw;
    if (!gene_ok(B, g, G, dcnt, &o, &len, &nw)) return;
    if (lane == 0) B.nwin[g] = nw;
    if (nw > kMvWaveCap) {
        if (lane == 0) {
            const uint64_t item = (static_cast<uint64_t>(t) << 32) | g;
            const uint32_t c = nw > kMvSortCap ? 0u : (nw <= kMvThreads * 8 ? 1u : (nw <= kMvThreads * 16 ? 2u : 3u));
            if (c == 0) long_list[atomicAdd(&counters[0], 1u)] = item;
            else mid_list[(c - 1) * stride + atomicAdd(&counters[c], 1u)] = item;
        }
        return;
    }
    uint8_t *sym = sym_all[w];
    // rounds of 4 residues per lane, the 4 loads issued before any is used
    for (uint32_t base = 0; base < len; base += 4 * kWave) {
        uint32_t res[4];
#pragma unroll
        for (uint32_t it = 0; it < 4; ++it) {
            const uint32_t p = base + lane + it * kWave;
            res[it] = p < len ? load_global(B.res + o + p) : 'A';
        }
#pragma unroll
        for (uint32_t it = 0; it < 4; ++it) {
            const uint32_t p = base + lane + it * kWave;
            if (p >= len) continue;
            uint32_t x = sym_in(res[it], B.bits);
            if (x == kInvalidSym) {
                raise_status(B.status, PDP_E_ALPHABET, 0, o + p);
                x = 0;
            }
            sym[p] = static_cast<uint8_t>(x);
        }
    }
    wave_lds_sync();
    uint32_t total;
    if (B.bits * B.k <= 32) {  // uniform per wave
        if (nw <= kWave * 4) mv_wave_gene<4, uint32_t, false, NARROW>(B, sym, hp_all[w], o, nw, &total);
        else if (nw <= kWave * 8) mv_wave_gene<8, uint32_t, false, NARROW>(B, sym, hp_all[w], o, nw, &total);
        else mv_wave_gene<16, uint32_t, false, NARROW>(B, sym, hp_all[w], o, nw, &total);
    } else if (base20_keys(B)) {
        if (nw <= kWave * 4) mv_wave_gene<4, uint32_t, true, NARROW>(B, sym, hp_all[w], o, nw, &total);
        else if (nw <= kWave * 8) mv_wave_gene<8, uint32_t, true, NARROW>(B, sym, hp_all[w], o, nw, &total);
        else mv_wave_gene<16, uint32_t, true, NARROW>(B, sym, hp_all[w], o, nw, &total);
    } else {
        if constexpr (!NARROW) {
            if (nw <= kWave * 4) mv_wave_gene<4, uint64_t, false, false>(B, sym, hp_all[w], o, nw, &total);
            else if (nw <= kWave * 8) mv_wave_gene<8, uint64_t, false, false>(B, sym, hp_all[w], o, nw, &total);
            else mv_wave_gene<16, uint64_t, false, false>(B, sym, hp_all[w], o, nw, &total);
        }
    }
    if (lane == 0) dcnt[G] = total;
}

// The smaller or the larger of two keys.
__device__ __forceinline__ uint32_t keep(uint32_t a, uint32_t b, bool smaller) { return pick(a, b, smaller ? 0u : ~0u); }
__device__ __forceinline__ uint64_t keep(uint64_t a, uint64_t b, bool smaller) { return (a < b) == smaller ? a : b; }

// Ascending bitonic sort of kMvThreads * E keys by one work-group, E per thread in blocked
// order (thread t holds elements t*E .. t*E+E-1): comparators inside a thread swap
// registers, those inside a wave pair lanes by shuffles, and only those across waves go
// through LDS (xch: kMvThreads * E keys), so a stage costs a barrier only when its stride
// spans waves.  Contains barriers; every thread of the work-group must call it.
template <uint32_t E, typename K>
__device__ __forceinline__ void block_bitonic_sort(K (&key)[E], K *xch) {
    constexpr uint32_t N = kMvThreads * E;
    const uint32_t t = threadIdx.x;
    for (uint32_t size = 2; size <= N; size <<= 1) {
        for (uint32_t j = size >> 1; j >= kWave * E; j >>= 1) {  // partner in another wave
            const uint32_t lj = j / E;
#pragma unroll
            for (uint32_t e = 0; e < E; ++e) xch[e * kMvThreads + t] = key[e];
            __syncthreads();
            const bool keep_min = ((t & lj) == 0) == ((t * E & size) == 0);  // size > E: the same for all e
#pragma unroll
            for (uint32_t e = 0; e < E; ++e) key[e] = keep(key[e], xch[e * kMvThreads + (t ^ lj)], keep_min);
            __syncthreads();
        }
        for (uint32_t j = min(size >> 1, kWave * E / 2); j >= E; j >>= 1) {  // partner lane in this wave
            const uint32_t lj = j / E;
            const bool keep_min = ((t & lj) == 0) == ((t * E & size) == 0);
#pragma unroll
            for (uint32_t e = 0; e < E; ++e) key[e] = keep(key[e], __shfl_xor(key[e], lj, kWave), keep_min);
        }
#pragma unroll
        for (uint32_t j = E / 2; j > 0; j >>= 1) {  // partner in this thread's registers
            if (j >= size) continue;
#pragma unroll
            for (uint32_t e = 0; e < E; ++e) {
                if (e & j) continue;
                const bool asc = ((t * E + e) & size) == 0;
                const K a = key[e], b = key[e | j];
                key[e] = keep(a, b, asc);
                key[e | j] = keep(a, b, !asc);
            }
        }
    }
}

// Genes queued by k_mv_wave with more windows than a wave sorts, up to kMvThreads * E: one
// work-group per gene.  The gene's symbols go to LDS, every thread encodes E consecutive
// windows (one new letter per window), the work-group sorts the codes in registers, and
// run heads ranked by a work-group scan give the multiplicity vector.  The symbols, the
// sort's exchange area and the head positions share one LDS array.
// One queued gene: len letters at offset o, nw <= kMvThreads * E windows; K as in the wave kernel.
template <uint32_t E, typename K, bool B20, bool NARROW>
__device__ __forceinline__ void mid_gene(const DevBuild &B, uint32_t G, uint64_t o, uint32_t len, uint32_t nw,
                                         uint64_t *xch64, K *s_last, uint32_t *tmp, uint32_t *__restrict__ dcnt) {
    const uint32_t tid = threadIdx.x, lane = lane_id(), w = tid / kWave;
    const uint32_t k = B.k, bits = B.bits;
    uint8_t *sym = reinterpret_cast<uint8_t *>(xch64);
    uint16_t *hp = reinterpret_cast<uint16_t *>(xch64);
    K *xch = reinterpret_cast<K *>(xch64);
    for (uint32_t base = 0; base < len; base += 4 * kMvThreads) {  // 4 loads in flight per thread
        uint32_t res[4];
#pragma unroll
        for (uint32_t it = 0; it < 4; ++it) {
            const uint32_t p = base + it * kMvThreads + tid;
            res[it] = p < len ? load_global(B.res + o + p) : 'A';
        }
#pragma unroll
        for (uint32_t it = 0; it < 4; ++it) {
            const uint32_t p = base + it * kMvThreads + tid;
            if (p >= len) continue;
            uint32_t x = sym_in(res[it], bits);
            if (x == kInvalidSym) {
                raise_status(B.status, PDP_E_ALPHABET, 0, o + p);
                x = 0;
            }
            sym[p] = static_cast<uint8_t>(x);
        }
    }
    __syncthreads();
    K key[E];
    window_keys<E, K, B20>(sym, tid * E, nw, k, bits, key);
    __syncthreads();  // the symbols are read before the sort overwrites them
    block_bitonic_sort<E, K>(key, xch);
    if (lane == kWave - 1) s_last[w] = key[E - 1];
    K before = __shfl_up(key[E - 1], 1, kWave);
    __syncthreads();
    if (lane == 0 && w > 0) before = s_last[w - 1];
    uint32_t hmask = 0, nh = 0;
#pragma unroll
    for (uint32_t e = 0; e < E; ++e) {
        const uint32_t i = tid * E + e;
        const K prev = e ? key[e - 1] : before;
        const bool h = i < nw && (i == 0 || key[e] != prev);
        hmask |= static_cast<uint32_t>(h) << e;
        nh += h;
    }
    uint32_t total;
    const uint32_t r0 = block_exclusive_scan<kMvThreads>(nh, tmp, &total);
    uint32_t *slot_cnt = B.slot_cnt + o;
    if constexpr (NARROW) {
        // as in the wave kernel: the keys back through LDS, so that the stores are whole lines; the
        // wave's first rank comes from the scan
        hp = reinterpret_cast<uint16_t *>(xch + kMvThreads * E);
#pragma unroll
        for (uint32_t e = 0; e < E; ++e) xch[tid * E + e] = key[e];
        uint32_t r = __shfl(r0, 0, kWave);
        __syncthreads();
        uint32_t *slot_key = reinterpret_cast<uint32_t *>(B.slot_code) + o;
        for (uint32_t q = 0; q < E; ++q) {
            const uint32_t i = w * kWave * E + q * kWave + lane;
            const K c = xch[i];
            const bool head = i < nw && (i == 0 || c != xch[i - 1]);
            const uint64_t mask = __ballot(head);
            const uint32_t at = r + mask_below(mask);
            if (head) {
                hp[at] = static_cast<uint16_t>(i);
                store_global(slot_key + at, c);
            }
            r += static_cast<uint32_t>(__popcll(mask));
        }
        if (tid == 0) hp[total] = static_cast<uint16_t>(nw);
        __syncthreads();
        for (uint32_t x = tid; x < total; x += kMvThreads)
            store_global(slot_cnt + x, static_cast<uint32_t>(hp[x + 1]) - hp[x]);
    } else {
        uint32_t r = r0;
#pragma unroll
        for (uint32_t e = 0; e < E; ++e)
            if ((hmask >> e) & 1u) hp[r++] = static_cast<uint16_t>(tid * E + e);
        if (tid == 0) hp[total] = static_cast<uint16_t>(nw);
        __syncthreads();
        uint64_t *slot_code = B.slot_code + o;
        r = r0;
#pragma unroll
        for (uint32_t e = 0; e < E; ++e) {
            if (!((hmask >> e) & 1u)) continue;
            store_global(slot_code + r, key_code<B20>(key[e], k));
            store_global(slot_cnt + r, static_cast<uint32_t>(hp[r + 1]) - hp[r]);
            ++r;
        }
    }
    if (tid == 0) dcnt[G] = total;
    __syncthreads();  // LDS takes the next gene
}

// One queued gene of at most kMvThreads * E windows.  xch: mid_words<E, NARROW> words.
template <uint32_t E, bool NARROW>
constexpr uint32_t mid_words = NARROW ? kMvThreads * E * 3 / 4 + 1 : kMvThreads * E;  // NARROW: N keys, N + 1 head positions
template <uint32_t E, bool NARROW>
__device__ __forceinline__ void mid_item(const DevBuild *__restrict__ table, uint64_t item, uint64_t *xch, uint64_t *s_last,
                                         uint32_t *tmp, uint32_t *__restrict__ dcnt) {
    constexpr uint32_t N = kMvThreads * E;
    static_assert(N + kKMaxAll <= 6 * N && N + 1 <= 4 * N && N <= 65535, "symbols and u16 head positions fit");
    const DevBuild &B = table[item >> 32];
    const uint32_t g = static_cast<uint32_t>(item);
    const uint64_t o = B.off[g];
    const uint32_t len = static_cast<uint32_t>(B.off[g + 1] - o);
    const uint32_t nw = len - B.k + 1;  // k_mv_wave queued this gene for nw <= kMvThreads * E
    if (B.bits * B.k <= 32) {  // uniform per work-group
        mid_gene<E, uint32_t, false, NARROW>(B, B.gene_base + g, o, len, nw, xch, reinterpret_cast<uint32_t *>(s_last), tmp, dcnt);
    } else if (base20_keys(B)) {
        mid_gene<E, uint32_t, true, NARROW>(B, B.gene_base + g, o, len, nw, xch, reinterpret_cast<uint32_t *>(s_last), tmp,
                                    dcnt);
    } else {
        if constexpr (!NARROW) mid_gene<E, uint64_t, false, false>(B, B.gene_base + g, o, len, nw, xch, s_last, tmp, dcnt);
    }
}

// The genes of up to 2048 windows (many, in a build of nucleotide genes).
template <bool NARROW>
__global__ __launch_bounds__(kMvThreads) void k_mv_mid(const DevBuild *__restrict__ table, uint32_t *__restrict__ dcnt,
                                                       const uint64_t *__restrict__ list,
                                                       const uint32_t *__restrict__ counters) {
    __shared__ uint64_t xch[mid_words<8, NARROW>];
    __shared__ uint64_t s_last[kMvWaves];
    __shared__ uint32_t tmp[kMvWaves + 1];
    const uint32_t n_items = counters[1];
    for (uint32_t li = blockIdx.x; li < n_items; li += gridDim.x) mid_item<8, NARROW>(table, list[li], xch, s_last, tmp, dcnt);
}

// Genes with more windows than fit in LDS: same steps, codes sorted in global memory.
template <bool NARROW>
__device__ __forceinline__ void long_item(const DevBuild *__restrict__ table, uint64_t item, uint32_t *tmp,
                                          uint32_t *__restrict__ dcnt) {
    const uint32_t tid = threadIdx.x;
    const DevBuild &B = table[item >> 32];
    const uint32_t g = static_cast<uint32_t>(item);
    const uint32_t k = B.k;
    const uint64_t o = B.off[g];
    const uint32_t nw = static_cast<uint32_t>(B.off[g + 1] - o - k + 1);
    uint64_t *w = B.long_tmp + o;
    for (uint64_t p = tid; p < nw + k - 1; p += kMvThreads)
        if (sym_in(B.res[o + p], B.bits) == kInvalidSym) raise_status(B.status, PDP_E_ALPHABET, 0, o + p);
    for (uint32_t p = tid; p < nw; p += kMvThreads) {
        uint64_t c = 0;
        for (uint32_t j = 0; j < k; ++j) {
            uint32_t s = sym_in(B.res[o + p + j], B.bits);
            c = (c << B.bits) | (s == kInvalidSym ? 0u : s);
        }
        w[p] = c;
    }
    __syncthreads();
    wg_network_sort(nw, [&](uint32_t lo, uint32_t hi) {
        const uint64_t a = w[lo], b = w[hi];
        if (b < a) {
            w[lo] = b;
            w[hi] = a;
        }
    });
    uint32_t base = 0;
    for (uint32_t c0 = 0; c0 < nw; c0 += kMvThreads) {
        const uint32_t i = c0 + tid;
        const bool head = i < nw && (i == 0 || w[i] != w[i - 1]);
        uint32_t total;
        const uint32_t r = block_exclusive_scan<kMvThreads>(head ? 1u : 0u, tmp, &total);
        if (head) {
            const uint64_t c = w[i];
            uint32_t end = i + 1;
            while (end < nw && w[end] == c) ++end;
            if constexpr (NARROW) reinterpret_cast<uint32_t *>(B.slot_code)[o + base + r] = code_to_key(B, c);
            else B.slot_code[o + base + r] = c;
            B.slot_cnt[o + base + r] = end - i;
        }
        base += total;
    }
    if (tid == 0) dcnt[B.gene_base + g] = base;
    __syncthreads();
}

// The longer genes of all classes in one launch, the longest first (a launch per class cost small
// builds 4.5 us each, and the classes of one nucleotide genome, 27 and 45 us, ran one after another).
template <bool NARROW>
__global__ __launch_bounds__(kMvThreads) void k_mv_rest(const DevBuild *__restrict__ table, uint32_t *__restrict__ dcnt,
                                                        const uint64_t *__restrict__ mid_list, uint32_t stride,
                                                        const uint64_t *__restrict__ long_list,
                                                        const uint32_t *__restrict__ counters) {
    __shared__ uint64_t xch[mid_words<32, NARROW>];
    __shared__ uint64_t s_last[kMvWaves];
    __shared__ uint32_t tmp[kMvWaves + 1];
    const uint32_t n_long = counters[0], n32 = counters[3], n16 = counters[2];
    for (uint32_t li = blockIdx.x; li < n_long + n32 + n16; li += gridDim.x) {  // uniform per work-group
        if (li < n_long) long_item<NARROW>(table, long_list[li], tmp, dcnt);
        else if (li < n_long + n32) mid_item<32, NARROW>(table, mid_list[2 * stride + li - n_long], xch, s_last, tmp, dcnt);
        else mid_item<16, NARROW>(table, mid_list[stride + li - n_long - n32], xch, s_last, tmp, dcnt);
    }
}

// One wave per gene: CSR offset of the gene and its vector moved into place.  For the index every
// entry leaves its record (REC: key and gene | count << 16, 8 bytes) or its gene, in the order of
// all genomes' entries.  NARROW: the slots hold 32-bit keys.  Bound by memory.
template <bool NARROW, bool REC>
__global__ __launch_bounds__(kWave) void k_mv_compact(const DevBuild *__restrict__ table, uint32_t n_genomes,
                                                      const uint32_t *__restrict__ gptr, uint32_t *__restrict__ ent_gene,
                                                      uint2 *__restrict__ ent_rec) {
    const uint32_t G = blockIdx.x;
    const DevBuild &B = table[find_genome_by_gene(table, n_genomes, G)];
    const uint32_t g = G - B.gene_base;
    const uint64_t o = B.off[g];
    const uint32_t base = gptr[B.gene_base];
    const uint32_t p = gptr[G] - base;
    const uint32_t d = gptr[G + 1] - gptr[G];
    if (threadIdx.x == 0) {
        B.mv_ptr[g] = p;
        if (g + 1 == B.n_genes) B.mv_ptr[g + 1] = p + d;
    }
    const uint32_t *slot_key = reinterpret_cast<const uint32_t *>(B.slot_code) + o;
    constexpr uint32_t U = 4;  // entries a thread has in flight
    for (uint32_t e0 = threadIdx.x; e0 < d; e0 += U * kWave) {
        uint64_t c[U];
        uint32_t n[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t e = e0 + u * kWave;
            if (e >= d) continue;
            if constexpr (NARROW) c[u] = load_global(slot_key + e);
            else c[u] = load_global(B.slot_code + o + e);
            n[u] = load_global(B.slot_cnt + o + e);
        }
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t e = e0 + u * kWave;
            if (e >= d) continue;
            if constexpr (NARROW) store_global(B.mv_code + p + e, key_to_code(B, static_cast<uint32_t>(c[u])));
            else store_global(B.mv_code + p + e, c[u]);
            store_global(B.mv_cnt + p + e, n[u]);
            if constexpr (REC) ent_rec[base + p + e] = make_uint2(static_cast<uint32_t>(c[u]), g | (n[u] << 16));
            else ent_gene[base + p + e] = g;
        }
    }
}


__device__ __forceinline__ uint32_t find_genome_by_block(const DevBuild *t, uint32_t n, uint32_t blk) {
    uint32_t lo = 0, hi = n - 1;
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) >> 1;
        if (t[mid].blk_base <= blk) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

__device__ __forceinline__ uint32_t find_genome_by_bin(const DevBuild *t, uint32_t n, uint32_t bin) {
    uint32_t lo = 0, hi = n - 1;
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) >> 1;
        if (t[mid].bin_base <= bin) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Block j's entries [j * blk, ...) of a genome: genome-local range, clipped to the genome's entry count.
__device__ __forceinline__ void block_range(const DevBuild &B, const uint32_t *gptr, uint32_t j, uint32_t *e0,
                                            uint32_t *e1, uint32_t *gbase) {
    const uint32_t base = gptr[B.gene_base];
    const uint32_t E = gptr[B.gene_base + B.n_genes] - base;
    *gbase = base;
    *e0 = min(E, j * B.blk);
    *e1 = min(E, (j + 1) * B.blk);
}

// Bucket of an entry: from its 32-bit key (REC) or its code.
template <bool REC>
__device__ __forceinline__ uint32_t entry_bucket(const DevBuild &B, uint64_t c) {
    if constexpr (REC)
        if (base20_keys(B)) return static_cast<uint32_t>(c) / 8000u;  // 20^3: the last three letters
    return bucket_of(c, B.k, B.lead, B.bits);
}

// One work-group per block of entries: coarse-bin histogram in LDS, added to the genome's
// bin totals with one global atomic per non-empty bin.
template <bool REC>
__global__ __launch_bounds__(256) void k_ix_hist(const DevBuild *__restrict__ table, uint32_t n_genomes,
                                                 const uint32_t *__restrict__ gptr, const uint2 *__restrict__ ent_rec,
                                                 uint32_t *__restrict__ bintot, uint32_t total_bins,
                                                 uint32_t *__restrict__ binoff, uint32_t *__restrict__ done) {
    extern __shared__ uint32_t h[];
    __shared__ uint32_t s_t, s_last;
    __shared__ uint32_t s_tmp[256 / kWave + 1];
    if (threadIdx.x == 0) s_t = find_genome_by_block(table, n_genomes, blockIdx.x);
    __syncthreads();
    const DevBuild &B = table[s_t];
    const uint32_t j = blockIdx.x - B.blk_base;
    for (uint32_t i = threadIdx.x; i < B.nh; i += blockDim.x) h[i] = 0;
    __syncthreads();
    uint32_t e0, e1, gbase;
    block_range(B, gptr, j, &e0, &e1, &gbase);
    // rounds of kIxBatch entries per thread: the loads of a round are issued before its atomics
    for (uint32_t base = e0; base < e1; base += kIxBatch * 256) {
        uint64_t c[kIxBatch];
#pragma unroll
        for (uint32_t q = 0; q < kIxBatch; ++q) {
            const uint32_t e = base + q * 256 + threadIdx.x;
            if constexpr (REC) c[q] = load_global(reinterpret_cast<const uint32_t *>(ent_rec + gbase + min(e, e1 - 1)));
            else c[q] = e < e1 ? load_global(B.mv_code + e) : 0ull;
        }
#pragma unroll
        for (uint32_t q = 0; q < kIxBatch; ++q)
            if (base + q * 256 + threadIdx.x < e1) atomicAdd(&h[entry_bucket<REC>(B, c[q]) >> B.hshift], 1u);
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < B.nh; i += blockDim.x)
        if (h[i]) atomicAdd(&bintot[B.bin_base + i], h[i]);
    if (!binoff) return;
    // few bins: the block that ends last scans the totals into every bin's range
    if (!last_group(done, &s_last)) return;
    uint32_t carry = 0;
    for (uint32_t b0 = 0; b0 < total_bins; b0 += 256 * 8) {
        uint32_t v[8], sum = 0;
#pragma unroll
        for (uint32_t q = 0; q < 8; ++q) {
            const uint32_t i = b0 + threadIdx.x * 8 + q;
            v[q] = i < total_bins ? __hip_atomic_load(&bintot[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
            sum += v[q];
        }
        uint32_t all;
        uint32_t run = carry + block_exclusive_scan<256>(sum, s_tmp, &all);
        carry += all;
#pragma unroll
        for (uint32_t q = 0; q < 8; ++q) {
            const uint32_t i = b0 + threadIdx.x * 8 + q;
            if (i < total_bins) binoff[i] = run;
            run += v[q];
        }
    }
    if (threadIdx.x == 0) binoff[total_bins] = carry;
}

__device__ __forceinline__ uint64_t rec_code(const uint4 &r) { return (static_cast<uint64_t>(r.y) << 32) | r.x; }
__device__ __forceinline__ uint32_t rec_gene(const uint4 &r) { return r.z; }
__device__ __forceinline__ uint32_t rec_cnt(const uint4 &r) { return r.w; }
__device__ __forceinline__ uint64_t rec_code(const uint2 &r) { return r.x; }
__device__ __forceinline__ uint32_t rec_gene(const uint2 &r) { return r.y & 0xFFFFu; }
__device__ __forceinline__ uint32_t rec_cnt(const uint2 &r) { return r.y >> 16; }
// An index record in the form a bin sort keeps in LDS: uint4 = (code low, code high, gene,
// count), or, when every genome of the build has 32-bit keys (codes of at most 32 bits, or
// base-20 values: base20_keys) and at most 65536 genes, uint2 = (key, gene | count << 16):
// half the LDS, more work-groups per CU.  A base-20 key orders records as the code does.
// The 5-bit code of a record.
__device__ __forceinline__ uint64_t rec_code5(const DevBuild &, const uint4 &r) { return rec_code(r); }
__device__ __forceinline__ uint64_t rec_code5(const DevBuild &B, const uint2 &r) {
    return base20_keys(B) ? base20_to_code(r.x, B.k) : static_cast<uint64_t>(r.x);
}

constexpr uint32_t kIxPlaceThreads = 1024;  // a placement work-group: its block of entries in registers, 16 per thread (2 in small builds)

// Same blocks: each entry goes to its bin's range.  The block counts its entries per bin in
// LDS (every entry's rank among the block's entries of its bin comes back from the LDS
// atomic), takes a run of each bin's range with one global atomic on the bin's remaining
// count (binoff holds the scanned totals; the runs of a bin are handed out from its end),
// and writes each entry at its run start plus its rank, in the record form R the bin sort
// keeps (8 bytes when the build allows it, so the scattered stores and the sort's loads move
// half the bytes).  The order inside a bin depends on scheduling; k_ix_sort_bin sorts every
// bin completely.  STAGE: the block's records go through LDS in the order of their bins first
// (128 KB, so one work-group of 16 waves per CU instead of two), so that a wave's store covers the few
// lines of its runs instead of 64 partial ones, which bound it: 1.53 GB written for 0.55 GB of records on
// 50 genomes.  450 -> 295 us there, 10 x 3000 genes 81 -> 60, nucleotides 292 -> 169, one nucleotide
// genome of 220 blocks 47 -> 32.  (With bins of 512 entries, runs of 6.5 records, it lost.)
template <typename R, uint32_t kIxPerThread, bool STAGE>
__global__ __launch_bounds__(kIxPlaceThreads) void k_ix_place(const DevBuild *__restrict__ table, uint32_t n_genomes,
                                                  const uint32_t *__restrict__ gptr, const uint32_t *__restrict__ binoff,
                                                  uint32_t *__restrict__ bintot, const uint32_t *__restrict__ ent_gene,
                                                  const uint2 *__restrict__ ent_rec) {
    constexpr bool REC = sizeof(R) == 8;
    extern __shared__ __align__(8) uint32_t cur[];
    __shared__ uint32_t s_t;
    if (threadIdx.x == 0) s_t = find_genome_by_block(table, n_genomes, blockIdx.x);
    __syncthreads();
    const DevBuild &B = table[s_t];
    const uint32_t j = blockIdx.x - B.blk_base;
    for (uint32_t i = threadIdx.x; i < B.nh; i += blockDim.x) cur[i] = 0;
    __syncthreads();
    uint32_t e0, e1, gbase;
    block_range(B, gptr, j, &e0, &e1, &gbase);
    if (e0 == e1) return;  // uniform
    using Key = typename std::conditional<REC, uint32_t, uint64_t>::type;
    Key c[kIxPerThread];
    uint32_t second[kIxPerThread];  // REC: gene and count
    uint32_t rank[kIxPerThread];
#pragma unroll
    for (uint32_t q = 0; q < kIxPerThread; ++q) {
        const uint32_t e = e0 + q * kIxPlaceThreads + threadIdx.x;
        if constexpr (REC) {
            const uint64_t r = load_global(reinterpret_cast<const uint64_t *>(ent_rec + gbase + min(e, e1 - 1)));
            c[q] = static_cast<uint32_t>(r);
            second[q] = static_cast<uint32_t>(r >> 32);
        } else {
            c[q] = e < e1 ? load_global(B.mv_code + e) : 0ull;
        }
    }
#pragma unroll
    for (uint32_t q = 0; q < kIxPerThread; ++q)
        if (e0 + q * kIxPlaceThreads + threadIdx.x < e1) rank[q] = atomicAdd(&cur[entry_bucket<REC>(B, c[q]) >> B.hshift], 1u);
    __syncthreads();
    const uint32_t gstart = binoff[B.bin_base];  // the genome's first entry in the scanned order
    if constexpr (STAGE) {
        static_assert(REC, "staged records are words");
        __shared__ uint32_t s_tmp[kIxPlaceThreads / kWave + 1];
        uint64_t *rec = reinterpret_cast<uint64_t *>(cur + ((B.nh + 1) & ~1u));
        const uint32_t per = (B.nh + kIxPlaceThreads - 1) / kIxPlaceThreads, b0 = threadIdx.x * per;
        uint32_t sum = 0, total;
        for (uint32_t b = 0; b < per && b0 + b < B.nh; ++b) sum += cur[b0 + b];
        uint32_t at = block_exclusive_scan<kIxPlaceThreads>(sum, s_tmp, &total);  // contains barriers
        uint32_t run[kIxMaxBins / kIxPlaceThreads];  // from a place in the block to its place in the genome
#pragma unroll
        for (uint32_t b = 0; b < kIxMaxBins / kIxPlaceThreads; ++b) {
            if (b >= per || b0 + b >= B.nh) continue;
            const uint32_t i = b0 + b, n = cur[i];
            cur[i] = at;
            run[b] = n ? binoff[B.bin_base + i] - gstart + atomicSub(&bintot[B.bin_base + i], n) - n - at : 0u;
            at += n;
        }
        __syncthreads();
#pragma unroll
        for (uint32_t q = 0; q < kIxPerThread; ++q)
            if (e0 + q * kIxPlaceThreads + threadIdx.x < e1)
                rec[cur[entry_bucket<REC>(B, c[q]) >> B.hshift] + rank[q]] = (static_cast<uint64_t>(second[q]) << 32) | c[q];
        __syncthreads();
#pragma unroll
        for (uint32_t b = 0; b < kIxMaxBins / kIxPlaceThreads; ++b)
            if (b < per && b0 + b < B.nh) cur[b0 + b] = run[b];
        __syncthreads();
#pragma unroll
        for (uint32_t q = 0; q < kIxPerThread; ++q) {
            const uint32_t i = q * kIxPlaceThreads + threadIdx.x;
            if (i >= e1 - e0) continue;
            const uint64_t r = rec[i];
            store_global(reinterpret_cast<uint64_t *>(B.ix_tmp) + (cur[entry_bucket<REC>(B, static_cast<uint32_t>(r)) >> B.hshift] + i), r);
        }
        return;
    }
    for (uint32_t i = threadIdx.x; i < B.nh; i += blockDim.x) {
        const uint32_t n = cur[i];
        if (n) cur[i] = binoff[B.bin_base + i] - gstart + atomicSub(&bintot[B.bin_base + i], n) - n;
    }
    __syncthreads();
    if constexpr (REC) {
#pragma unroll
        for (uint32_t q = 0; q < kIxPerThread; ++q) {
            if (e0 + q * kIxPlaceThreads + threadIdx.x >= e1) continue;
            const uint32_t pos = cur[entry_bucket<REC>(B, c[q]) >> B.hshift] + rank[q];
            // one 64-bit word, through a global (not flat) store
            store_global(reinterpret_cast<uint64_t *>(B.ix_tmp) + pos, (static_cast<uint64_t>(second[q]) << 32) | c[q]);
        }
    } else {
        constexpr uint32_t kRound = kIxPerThread < kIxBatch ? kIxPerThread : kIxBatch;
        for (uint32_t q0 = 0; q0 < kIxPerThread; q0 += kRound) {
            uint32_t gn[kRound], ct[kRound];
#pragma unroll
            for (uint32_t q = 0; q < kRound; ++q) {
                const uint32_t e = e0 + (q0 + q) * kIxPlaceThreads + threadIdx.x;
                const bool v = e < e1;
                gn[q] = v ? ent_gene[gbase + e] : 0u;
                ct[q] = v ? load_global(B.mv_cnt + e) : 0u;
            }
#pragma unroll
            for (uint32_t q = 0; q < kRound; ++q) {
                if (e0 + (q0 + q) * kIxPlaceThreads + threadIdx.x >= e1) continue;
                const uint64_t code = c[q0 + q];
                const uint32_t pos = cur[entry_bucket<REC>(B, code) >> B.hshift] + rank[q0 + q];
                // one record per entry: a single scattered store instead of three
                B.ix_tmp[pos] = make_uint4(static_cast<uint32_t>(code), static_cast<uint32_t>(code >> 32), gn[q], ct[q]);
            }
        }
    }
}

__device__ __forceinline__ bool entry_less(uint64_t ca, uint32_t ga, uint64_t cb, uint32_t gb) {
    return ca < cb || (ca == cb && ga < gb);
}

template <typename CP, typename GP>
__device__ void sort_entries(CP code, GP gene, GP cnt, uint32_t n) {
    wg_network_sort(n, [&](uint32_t lo, uint32_t hi) {
        const uint64_t cl = code[lo], ch = code[hi];
        const uint32_t gl = gene[lo], gh = gene[hi];
        if (entry_less(ch, gh, cl, gl)) {
            code[lo] = ch;
            code[hi] = cl;
            gene[lo] = gh;
            gene[hi] = gl;
            const uint32_t t = cnt[lo];
            cnt[lo] = cnt[hi];
            cnt[hi] = t;
        }
    });
}

// Directory entries of buckets [b0, b1) from a bin sorted by code: the first entry of
// each bucket, found by binary search on the bucket of the codes.
template <typename CP>
__device__ void bin_directory(const DevBuild &B, CP code, uint32_t n, uint32_t lo, uint32_t b0, uint32_t b1) {
    for (uint32_t b = b0 + threadIdx.x; b < b1; b += blockDim.x) {
        uint32_t l = 0, r = n;
        while (l < r) {
            const uint32_t mid = (l + r) >> 1;
            if (bucket_of(code[mid], B.k, B.lead, B.bits) < b) l = mid + 1;
            else r = mid;
        }
        B.ix_dir[b] = lo + l;
    }
}

// Packed join key of an index entry: the code's trailing letters (the leading ones are
// the bucket) above the gene.
__device__ __forceinline__ uint32_t entry_key(const DevBuild &B, uint64_t code, uint32_t gene) {
    const uint32_t tb = B.bits * (B.k - B.lead);
    const uint64_t tail = tb ? code & ((1ull << tb) - 1) : 0ull;
    return static_cast<uint32_t>(tail << B.key_shift) | gene;
}

template <typename R>
__device__ __forceinline__ void put_entry(const DevBuild &B, uint32_t pos, const R &v) {
    const uint64_t c = rec_code5(B, v);
    const uint32_t g = rec_gene(v);
    store_global(B.ix_code + pos, c);
    store_global(B.ix_gene + pos, g);
    store_global(B.ix_cnt + pos, rec_cnt(v));
    if (B.key_shift) store_global(B.ix_key + pos, entry_key(B, c, g));
}
template <typename R>
__device__ __forceinline__ bool rec_less(const R &a, const R &b) {
    return entry_less(rec_code(a), rec_gene(a), rec_code(b), rec_gene(b));
}

// Work-group sort of index records (code, gene, count) in LDS by (code, gene).
template <typename R>
__device__ __forceinline__ void sort_recs(R *r, uint32_t n) {
    wg_network_sort(n, [&](uint32_t lo, uint32_t hi) {
        const R a = r[lo], b = r[hi];
        if (rec_less(b, a)) {
            r[lo] = b;
            r[hi] = a;
        }
    });
}

constexpr uint32_t kIxSmallBucket = 32;   // slots up to this size are ranked entry by entry
constexpr uint32_t kIxBigList = 64;       // larger slots a bin sorts one by one with the work-group
constexpr uint32_t kIxCuts = 32;          // parts of a bin past LDS that are laid out at a time
// A bin sort's work-group: LDS for 4096 records of 8 bytes or 1024 of 16, and twice as many slots.
template <typename R>
struct BinSort {
    static constexpr uint32_t kThreads = sizeof(R) == 8 ? 512 : 256;
    static constexpr uint32_t kPer = sizeof(R) == 8 ? 8 : 4;   // entries per thread
    static constexpr uint32_t kLds = kThreads * kPer;      // entries of a bin sorted in LDS
    static constexpr uint32_t kSlots = 2 * kLds;           // counting-sort slots of a bin (buckets x sub-slots)
    static constexpr uint32_t kWords = kSlots / 2 / kThreads;  // 16-bit slot counters, words per thread
    static constexpr uint32_t kWavesPerSimd = sizeof(R) == 8 ? 6 : 7;  // what the LDS allows
};

// Counting-sort slot of a code inside the bin starting at bucket b0: the bucket, then the
// next xb bits of the code, so slots ascend like codes.
__device__ __forceinline__ uint32_t bin_slot(const DevBuild &B, uint64_t code, uint32_t b0) {
    const uint32_t b = bucket_of(code, B.k, B.lead, B.bits) - b0;
    if (!B.xb) return b;
    const uint32_t sh = B.bits * (B.k - B.lead) - B.xb;
    return (b << B.xb) | (static_cast<uint32_t>(code >> sh) & ((1u << B.xb) - 1u));
}
// The same from a record: a base-20 key of a 7-mer gives its bucket (first 4 letters) and next
// letter directly.
__device__ __forceinline__ uint32_t rec_slot(const DevBuild &B, const uint4 &r, uint32_t b0) {
    return bin_slot(B, rec_code(r), b0);
}
__device__ __forceinline__ uint32_t rec_slot(const DevBuild &B, const uint2 &r, uint32_t b0) {
    if (!base20_keys(B)) return bin_slot(B, r.x, b0);
    const uint32_t b = r.x / 8000u - b0;  // 20^3: the last three letters
    return B.xb ? (b << B.xb) | (((r.x / 400u) % 20u) >> (5u - B.xb)) : b;
}

__device__ __forceinline__ uint32_t slot16(const uint32_t *w, uint32_t s) { return (w[s >> 1] >> ((s & 1u) * 16u)) & 0xFFFFu; }

// LDS of a bin sort's work-group.
template <typename R>
struct BinLds {
    R rec[BinSort<R>::kLds];
    uint32_t slot[BinSort<R>::kSlots / 2 + 1];  // two 16-bit counters, then starts, per word
    uint32_t big[kIxBigList];
    uint32_t tmp[BinSort<R>::kThreads / kWave + 1];
    uint32_t cut[kIxCuts + 1], pos[kIxCuts + 1];  // parts of a bin past LDS: first slot, entries before it
    uint32_t nbig, n, ncuts;
};

// The m records in registers (record q * kThreads + tid in r[q]), all of slots [c0, c0 + kSlots) of the bin from
// bucket b0 on, to the index from entry lo on, ordered by (code, gene): a counting sort by slot (LDS
// histogram, scan, scatter), then every entry finds its rank among its slot's entries and goes
// straight to its place.  Slots past kIxSmallBucket entries are sorted by the work-group first.
// L.slot (left holding the slots' starts) and L.nbig are zero before, with a barrier in between.
template <typename R>
__device__ __forceinline__ void bin_part(const DevBuild &B, const R (&r)[BinSort<R>::kPer], uint32_t m, uint32_t b0,
                                         uint32_t c0, uint32_t lo, BinLds<R> &L) {
    using S = BinSort<R>;
    constexpr uint32_t NT = S::kThreads, kIxPer = S::kPer;
    const uint32_t tid = threadIdx.x;
    uint32_t rank[kIxPer], bk[kIxPer];
#pragma unroll
    for (uint32_t q = 0; q < kIxPer; ++q) {
        if (q * NT + tid >= m) continue;
        const uint32_t b = rec_slot(B, r[q], b0) - c0, sh = (b & 1u) * 16u;
        bk[q] = b;
        rank[q] = (atomicAdd(&L.slot[b >> 1], 1u << sh) >> sh) & 0xFFFFu;
    }
    __syncthreads();
    {  // exclusive scan of the slot sizes
        uint32_t w[S::kWords], sum = 0;
#pragma unroll
        for (uint32_t q = 0; q < S::kWords; ++q) {
            w[q] = L.slot[tid * S::kWords + q];
            sum += (w[q] & 0xFFFFu) + (w[q] >> 16);
        }
        uint32_t total;
        uint32_t run = block_exclusive_scan<NT>(sum, L.tmp, &total);
#pragma unroll
        for (uint32_t q = 0; q < S::kWords; ++q) {
            const uint32_t b = (tid * S::kWords + q) * 2, n0 = w[q] & 0xFFFFu, n1 = w[q] >> 16;
            L.slot[tid * S::kWords + q] = run | ((run + n0) << 16);
            run += n0 + n1;
            for (uint32_t x = 0; x < 2; ++x)
                if ((x ? n1 : n0) > kIxSmallBucket) {
                    const uint32_t idx = atomicAdd(&L.nbig, 1u);
                    if (idx < kIxBigList) L.big[idx] = b + x;
                }
        }
        if (tid == 0) L.slot[S::kSlots / 2] = m;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t q = 0; q < kIxPer; ++q)
        if (q * NT + tid < m) L.rec[slot16(L.slot, bk[q]) + rank[q]] = r[q];
    __syncthreads();
    const uint32_t nbig = L.nbig;
    if (nbig > kIxBigList) {
        sort_recs(L.rec, m);
    } else {
        for (uint32_t j = 0; j < nbig; ++j) {  // uniform loop
            const uint32_t a = slot16(L.slot, L.big[j]);
            sort_recs(L.rec + a, slot16(L.slot, L.big[j] + 1) - a);
        }
    }
    for (uint32_t p = tid; p < m; p += NT) {
        const R v = L.rec[p];
        uint32_t at = p;
        const uint32_t b = rec_slot(B, v, b0) - c0, a = slot16(L.slot, b), e = slot16(L.slot, b + 1);
        if (e - a <= kIxSmallBucket && nbig <= kIxBigList) {
            at = a;
            for (uint32_t x = a; x < e; ++x) at += rec_less(L.rec[x], v);
        }
        put_entry(B, lo + at, v);
    }
}

// A record of the placement, through a global (not flat) load.
__device__ __forceinline__ uint2 load_rec(const uint2 *p) {
    const uint64_t w = load_global(reinterpret_cast<const uint64_t *>(p));
    return uint2{static_cast<uint32_t>(w), static_cast<uint32_t>(w >> 32)};
}
__device__ __forceinline__ uint4 load_rec(const uint4 *p) { return *p; }

// Slots [c, end) of a bin: end the largest so that their entries fit LDS, or c + 1 (start[x]: entries before
// slot x of nslot, n in all).
__device__ __forceinline__ uint32_t part_end(const uint32_t *start, uint32_t c, uint32_t nslot, uint32_t n, uint32_t cap) {
    uint32_t l = c + 1, h = nslot;
    while (l < h) {
        const uint32_t mid = (l + h + 1) >> 1;
        if ((mid < nslot ? start[mid] : n) - start[c] <= cap) l = mid;
        else h = mid - 1;
    }
    return l;
}

// A bin past LDS: its slots are counted (32-bit counters over the record array) and it goes through LDS in
// ranges of slots that fit, each picked out of the whole bin; only a single slot past LDS (equal k-mers in
// more genes than LDS holds) is sorted in place in global memory.
template <typename R>
__device__ __forceinline__ void bin_in_parts(const DevBuild &B, const R *tmp, uint32_t n, uint32_t lo, uint32_t b0, uint32_t nbb,
                                             BinLds<R> &L) {
    using S = BinSort<R>;
    constexpr uint32_t NT = S::kThreads, kPerScan = S::kSlots / NT;
    static_assert(S::kSlots * sizeof(uint32_t) <= sizeof(L.rec), "the counters fit the record array");
    const uint32_t tid = threadIdx.x, nslot = nbb << B.xb;
    uint32_t *start = reinterpret_cast<uint32_t *>(L.rec);
    for (uint32_t from = 0; from < nslot;) {  // kIxCuts parts at a time; uniform
        for (uint32_t i = tid; i < S::kSlots; i += NT) start[i] = 0;
        __syncthreads();
        for (uint32_t i = tid; i < n; i += NT) atomicAdd(&start[rec_slot(B, load_rec(tmp + i), b0)], 1u);
        __syncthreads();
        uint32_t c[kPerScan], sum = 0, total;
#pragma unroll
        for (uint32_t q = 0; q < kPerScan; ++q) {
            c[q] = start[tid * kPerScan + q];
            sum += c[q];
        }
        uint32_t run = block_exclusive_scan<NT>(sum, L.tmp, &total);  // contains barriers
#pragma unroll
        for (uint32_t q = 0; q < kPerScan; ++q) {
            start[tid * kPerScan + q] = run;
            run += c[q];
        }
        __syncthreads();
        if (from == 0)
            for (uint32_t b = tid; b < nbb; b += NT) store_global(B.ix_dir + b0 + b, lo + start[b << B.xb]);
        if (tid == 0) {
            uint32_t k = 0, x = from;
            for (; k < kIxCuts && x < nslot; ++k) {
                L.cut[k] = x;
                L.pos[k] = start[x];
                x = part_end(start, x, nslot, n, S::kLds);
            }
            L.cut[k] = x;
            L.pos[k] = x < nslot ? start[x] : n;
            L.ncuts = k;
        }
        __syncthreads();
        const uint32_t ncuts = L.ncuts;
        for (uint32_t k = 0; k < ncuts; ++k) {
            const uint32_t c0 = L.cut[k], c1 = L.cut[k + 1], at0 = lo + L.pos[k], m = L.pos[k + 1] - L.pos[k];
            const bool fits = m <= S::kLds;  // uniform
            if (m == 0) continue;
            __syncthreads();  // the record array is read before it takes the part
            if (tid == 0) {
                L.n = 0;
                L.nbig = 0;
            }
            for (uint32_t i = tid; i <= S::kSlots / 2; i += NT) L.slot[i] = 0;
            __syncthreads();
            for (uint32_t i0 = 0; i0 < n; i0 += NT) {
                R v{};
                bool in = i0 + tid < n;
                if (in) {
                    v = load_rec(tmp + i0 + tid);
                    const uint32_t x = rec_slot(B, v, b0);
                    in = x >= c0 && x < c1;
                }
                const uint64_t mask = __ballot(in);
                uint32_t at = 0;
                if (lane_id() == 0 && mask) at = atomicAdd(&L.n, static_cast<uint32_t>(__popcll(mask)));
                at = __shfl(at, 0, kWave) + mask_below(mask);
                if (!in) continue;
                if (fits) {
                    L.rec[at] = v;
                } else {
                    B.ix_code[at0 + at] = rec_code5(B, v);
                    B.ix_gene[at0 + at] = rec_gene(v);
                    B.ix_cnt[at0 + at] = rec_cnt(v);
                }
            }
            __syncthreads();
            if (fits) {
                R r[S::kPer];
#pragma unroll
                for (uint32_t q = 0; q < S::kPer; ++q) {
                    const uint32_t i = q * NT + tid;
                    r[q] = i < m ? L.rec[i] : R{};
                }
                __syncthreads();
                bin_part<R>(B, r, m, b0, c0, at0, L);
            } else {
                sort_entries(B.ix_code + at0, B.ix_gene + at0, B.ix_cnt + at0, m);
                if (B.key_shift)
                    for (uint32_t i = tid; i < m; i += NT)
                        B.ix_key[at0 + i] = entry_key(B, B.ix_code[at0 + i], B.ix_gene[at0 + i]);
            }
        }
        from = L.cut[ncuts];
        __syncthreads();
    }
}

// One work-group per coarse bin: its entries ordered by (code, gene) and the bin's part of
// the bucket directory.  Usual case: the bin fits LDS and its slots fit kSlots (bin_part, whose slot
// starts at the first slot of every bucket are the directory).  Letters are not used evenly, so some bins
// of large builds do not fit (bin_in_parts).  A bin of too many slots (tiny genomes) is sorted in LDS, or in
// place in global memory when it does not fit either.
// Bins of 1350 to 2700 8-byte records on average (50 genomes of 3000 to 5000 genes: 2176): sort 0.44 ms,
// placement 0.30 ms (0.45 before its records were staged).  With half of that 0.56 and 0.55 ms, with a
// quarter 0.87 and 0.70 ms, unstaged: the placement's runs per (block, bin) get shorter and the work-groups
// emptier.
template <typename R>
__global__ __launch_bounds__(BinSort<R>::kThreads, BinSort<R>::kWavesPerSimd) void k_ix_sort_bin(const DevBuild *__restrict__ table,
                                                                      uint32_t n_genomes,
                                                                      const uint32_t *__restrict__ off) {
    using S = BinSort<R>;
    constexpr uint32_t NT = S::kThreads, kIxPer = S::kPer;
    __shared__ BinLds<R> L;
    const uint32_t tid = threadIdx.x;
    const DevBuild &B = table[find_genome_by_bin(table, n_genomes, blockIdx.x)];
    const uint32_t h = blockIdx.x - B.bin_base;
    const uint32_t base = off[B.bin_base];
    const uint32_t lo = off[B.bin_base + h] - base;
    const uint32_t hi = off[B.bin_base + h + 1] - base;  // for the last bin: the next genome's start
    const uint32_t n = hi - lo;
    const uint32_t b0 = h << B.hshift;
    const uint32_t b1 = min(B.nb, (h + 1) << B.hshift);
    const uint32_t nbb = b1 - b0;
    const uint32_t nslot = nbb << B.xb;
    const R *tmp = reinterpret_cast<const R *>(B.ix_tmp) + lo;  // the placement wrote R records
    if (n <= S::kLds && nslot <= S::kSlots) {
        for (uint32_t i = tid; i <= S::kSlots / 2; i += NT) L.slot[i] = 0;
        if (tid == 0) L.nbig = 0;
        R r[kIxPer];
#pragma unroll
        for (uint32_t q = 0; q < kIxPer; ++q) {  // every load issued before the first atomic
            const uint32_t i = q * NT + tid;
            r[q] = i < n ? load_rec(tmp + i) : R{};
        }
        __syncthreads();
        bin_part<R>(B, r, n, b0, 0, lo, L);
        for (uint32_t b = tid; b < nbb; b += NT) store_global(B.ix_dir + b0 + b, lo + slot16(L.slot, b << B.xb));
    } else if (n <= S::kLds) {
        for (uint32_t i = tid; i < n; i += NT) L.rec[i] = tmp[i];
        __syncthreads();
        sort_recs(L.rec, n);
        for (uint32_t i = tid; i < n; i += NT) put_entry(B, lo + i, L.rec[i]);
        __syncthreads();
        bin_directory(B, B.ix_code + lo, n, lo, b0, b1);
    } else if (nslot <= S::kSlots) {
        bin_in_parts<R>(B, tmp, n, lo, b0, nbb, L);
    } else {
        for (uint32_t i = tid; i < n; i += NT) {
            const R v = tmp[i];
            B.ix_code[lo + i] = rec_code5(B, v);
            B.ix_gene[lo + i] = rec_gene(v);
            B.ix_cnt[lo + i] = rec_cnt(v);
        }
        __syncthreads();
        sort_entries(B.ix_code + lo, B.ix_gene + lo, B.ix_cnt + lo, n);
        if (B.key_shift)
            for (uint32_t i = tid; i < n; i += NT) B.ix_key[lo + i] = entry_key(B, B.ix_code[lo + i], B.ix_gene[lo + i]);
        bin_directory(B, B.ix_code + lo, n, lo, b0, b1);
    }
    if (h + 1 == B.nh && tid == 0) B.ix_dir[B.nb] = hi;
}

// ------------------------------------------------------------------ host

// Coarse-bin shift: bins of 2^s buckets holding at most `target` entries on average.
static uint32_t bin_shift(uint32_t nb, uint64_t cap, uint32_t target) {
    uint32_t s = 0;
    while ((uint64_t(nb) >> (s + 1)) > 0 && (cap << (s + 1)) <= uint64_t(nb) * target) ++s;
    while ((uint64_t(nb) >> s) > kIxMaxBins) ++s;  // keep the LDS histogram bounded
    return s;
}

// Bin shift s and sub-slot bits xb of one genome: a bin's counting sort goes by bucket and the leading bits
// of the next letter (amino acids, 5 bits) or two (nucleotides, 4 bits), all of them or as many as the
// slots hold, so that a slot holds few entries also where letters are frequent (2000 genes with the letters
// of proteins: 221 us by buckets alone, 138 so).
struct BinPlan {
    uint32_t s, xb;
};
static BinPlan bin_plan(uint32_t nb, uint64_t cap, uint32_t k, uint32_t alphabet, uint32_t target, uint32_t slots) {
    const AlphaSpec a = alpha_spec(alphabet);
    const uint32_t s = bin_shift(nb, cap, target);
    const uint32_t rest = k - lead_letters(k, alphabet);
    uint32_t xb = a.bits * std::min<uint32_t>(rest, a.bits == 2 ? 2u : 1u);
    while (xb && (1ull << (s + xb)) > slots) --xb;
    return {s, xb};
}

static BuildShape shape_of(const pdp_genome *g, const pdp_dict *const *d, uint32_t n) {
    BuildShape s{};
    s.n_genomes = n;
    for (uint32_t i = 0; i < n; ++i) {
        const uint64_t cap = g[i].n_residues + 1;
        const uint32_t nb = d[i]->n_buckets;
        const uint32_t sh = bin_shift(nb, cap, kIxBinTargetWide);  // the most bins a launch may choose
        const uint64_t nh = (uint64_t(nb) + (1ull << sh) - 1) >> sh;
        s.total_genes += g[i].n_genes;
        s.total_residues += cap;
        s.total_bins += nh;
    }
    return s;
}

uint64_t build_ws_bytes(const BuildShape &s) {
    const uint64_t A = 256;
    uint64_t b = 0;
    b += align_up(sizeof(DevBuild) * std::max<uint64_t>(s.n_genomes, 1), A);
    b += align_up(8 * s.total_residues, A);             // slot_code
    b += align_up(4 * s.total_residues, A);             // slot_cnt
    b += align_up(8 * s.total_residues, A);             // long_tmp
    b += align_up(4 * s.total_residues, A);             // ent_gene
    b += align_up(16 * s.total_residues, A);            // ix_tmp
    b += align_up(4 * (s.total_genes + 1), A);          // dcnt / gptr
    b += align_up(4 * (s.total_bins + 1), A);           // bin totals
    b += align_up(4 * (s.total_bins + 1), A);           // scanned bin offsets
    b += align_up(8 * (s.total_genes + 1), A);          // long_list
    b += align_up(3 * 8 * (s.total_genes + 1), A);      // mid_list: three size classes
    b += align_up(4 * kBuildCounters, A);               // counters
    const uint64_t np = std::max<uint64_t>(scan_partials(s.total_genes), scan_partials(s.total_bins));
    b += align_up(4 * np, A);
    return b;
}

BuildShape build_shape(const pdp_genome *g, const pdp_dict *const *d, uint32_t n) { return shape_of(g, d, n); }

BuildShape single_build_shape(uint32_t n_genes, uint64_t n_residues, uint32_t k, uint32_t alphabet) {
    pdp_genome g{};
    g.n_genes = n_genes;
    g.n_residues = n_residues;
    pdp_dict d{};
    d.k = k;
    d.alphabet = alphabet;
    d.n_buckets = n_buckets_for(k, alphabet);
    const pdp_dict *dp = &d;
    return shape_of(&g, &dp, 1);
}

hipError_t launch_dict_build_many(const pdp_genome *g, pdp_dict *const *d, uint32_t n, void *ws, hipStream_t s) {
    const BuildShape sh = shape_of(g, d, n);
    const uint64_t A = 256;
    char *p = static_cast<char *>(ws);
    auto take = [&](uint64_t bytes) {
        char *q = p;
        p += align_up(bytes, A);
        return q;
    };
    DevBuild *table = reinterpret_cast<DevBuild *>(take(sizeof(DevBuild) * std::max<uint64_t>(n, 1)));
    uint64_t *slot_code = reinterpret_cast<uint64_t *>(take(8 * sh.total_residues));
    uint32_t *slot_cnt = reinterpret_cast<uint32_t *>(take(4 * sh.total_residues));
    uint64_t *long_tmp = reinterpret_cast<uint64_t *>(take(8 * sh.total_residues));
    uint32_t *ent_gene = reinterpret_cast<uint32_t *>(take(4 * sh.total_residues));
    uint4 *ix_tmp = reinterpret_cast<uint4 *>(take(16 * sh.total_residues));
    uint32_t *dcnt = reinterpret_cast<uint32_t *>(take(4 * (sh.total_genes + 1)));
    uint32_t *bintot = reinterpret_cast<uint32_t *>(take(4 * (sh.total_bins + 1)));
    uint32_t *binoff = reinterpret_cast<uint32_t *>(take(4 * (sh.total_bins + 1)));
    uint64_t *long_list = reinterpret_cast<uint64_t *>(take(8 * (sh.total_genes + 1)));
    uint64_t *mid_list = reinterpret_cast<uint64_t *>(take(3 * 8 * (sh.total_genes + 1)));
    const uint32_t stride = static_cast<uint32_t>(sh.total_genes + 1);
    uint32_t *counters = reinterpret_cast<uint32_t *>(take(4 * kBuildCounters));
    const uint64_t np = std::max<uint64_t>(scan_partials(sh.total_genes), scan_partials(sh.total_bins));
    uint32_t *partials = reinterpret_cast<uint32_t *>(take(4 * np));

    // keys of 32 bits (codes, or base-20 values); records of 8 bytes when every gene index also fits
    // 16 bits and every multiplicity 16 bits (no long-gene dictionary)
    bool narrow = true, narrow_rec = true;
    for (uint32_t i = 0; i < n; ++i) {
        narrow &= alpha_spec(d[i]->alphabet).bits * d[i]->k <= 32 || (d[i]->alphabet == PDP_ALPHA_AMINO && d[i]->k == 7);
        narrow_rec &= g[i].n_genes <= 65536 && !(d[i]->flags & PDP_DICT_LONG_GENES);
    }
    narrow_rec &= narrow;
    // entries per placement block and per bin: large ones give each (block, bin) a longer run; builds
    // that leave the chip mostly idle take small blocks and bins.  One genome, small against large: 340,000
    // letters (1000 genes) 84 / 98 us, 510,000 94 / 104, 680,000 117 / 109, 1.46 million 187 / 129; k = 8
    // 102 / 119, 122 / 129, 137 / 143, 216 / 185; nucleotides 111 / 130, 121 / 130, 140 / 135, 223 / 180; six
    // genomes 79 / 101, 93 / 110, 98 / 113, 140 / 133.
    const bool small = sh.total_residues <= 40ull * kIxBlock;
    const uint32_t blk = small ? kIxBlockSmall : kIxBlock;
    const uint32_t target = narrow_rec && !small ? kIxBinTarget : kIxBinTargetWide;
    const uint32_t slots = narrow_rec ? BinSort<uint2>::kSlots : BinSort<uint4>::kSlots;
    uint32_t max_nh = 0;

    // descriptors, passed by value to a tiny kernel in chunks
    uint32_t total_bins = 0;
    for (uint32_t i = 0; i < n; ++i) {
        const uint32_t sh_i = bin_plan(d[i]->n_buckets, g[i].n_residues + 1, d[i]->k, d[i]->alphabet, target, slots).s;
        total_bins += static_cast<uint32_t>((uint64_t(d[i]->n_buckets) + (1ull << sh_i) - 1) >> sh_i);
    }
    uint64_t gene_base = 0, res_base = 0, blk_base = 0, bin_base = 0;
    for (uint32_t c0 = 0; c0 < n; c0 += kDescPerLaunch) {
        DescChunk ch{};
        ch.first = c0;
        ch.count = std::min<uint32_t>(kDescPerLaunch, n - c0);
        for (uint32_t j = 0; j < ch.count; ++j) {
            const pdp_genome &G = g[c0 + j];
            const pdp_dict &D = *d[c0 + j];
            DevBuild &B = ch.d[j];
            const uint64_t cap = G.n_residues + 1;
            B.res = G.residues;
            B.off = G.gene_off;
            B.n_residues = G.n_residues;
            B.n_genes = G.n_genes;
            B.k = D.k;
            B.nb = D.n_buckets;
            B.lead = D.lead;
            B.bits = alpha_spec(D.alphabet).bits;
            const BinPlan bp = bin_plan(D.n_buckets, cap, D.k, D.alphabet, target, slots);
            B.hshift = bp.s;
            B.xb = bp.xb;
            B.nh = static_cast<uint32_t>((uint64_t(D.n_buckets) + (1ull << B.hshift) - 1) >> B.hshift);
            B.blk = blk;
            B.nblk = static_cast<uint32_t>((cap + blk - 1) / blk);
            max_nh = std::max(max_nh, B.nh);
            B.gene_base = static_cast<uint32_t>(gene_base);
            B.blk_base = static_cast<uint32_t>(blk_base);
            B.bin_base = static_cast<uint32_t>(bin_base);
            B.nwin = D.nwin;
            B.mv_ptr = D.mv_ptr;
            B.mv_code = D.mv_code;
            B.mv_cnt = D.mv_cnt;
            B.ix_dir = D.ix_dir;
            B.ix_code = D.ix_code;
            B.ix_gene = D.ix_gene;
            B.ix_cnt = D.ix_cnt;
            B.ix_key = D.ix_key;
            B.key_shift = D.key_shift;
            B.max_windows = (D.flags & PDP_DICT_LONG_GENES) ? PDP_MAX_WINDOWS_LONG : PDP_MAX_WINDOWS;
            B.status = D.status;
            B.slot_code = slot_code + res_base;
            B.slot_cnt = slot_cnt + res_base;
            B.long_tmp = long_tmp + res_base;
            B.ix_tmp = ix_tmp + res_base;
            gene_base += G.n_genes;
            res_base += cap;
            blk_base += B.nblk;
            bin_base += B.nh;
        }
        const uint32_t init_grid = c0 ? 1u : std::min<uint32_t>(total_bins / 256 + 1, 1024);
        hipLaunchKernelGGL(k_build_init, dim3(init_grid), dim3(256), 0, s, table, ch, counters, bintot, total_bins);
        PDP_TRY(hipGetLastError());
    }
    const uint32_t tg = static_cast<uint32_t>(sh.total_genes);
    uint2 *ent_rec = reinterpret_cast<uint2 *>(long_tmp);  // free once the multiplicity vectors are in their slots
    const uint32_t total_blocks = static_cast<uint32_t>(blk_base);
    const uint32_t hist_lds = 4 * max_nh;
    if (tg > 0) {
        if (narrow)
            hipLaunchKernelGGL(k_mv_wave<true>, dim3((tg + kMvWaves - 1) / kMvWaves), dim3(kMvThreads), 0, s, table, n,
                               tg, dcnt, mid_list, long_list, stride, counters);
        else
            hipLaunchKernelGGL(k_mv_wave<false>, dim3((tg + kMvWaves - 1) / kMvWaves), dim3(kMvThreads), 0, s, table, n,
                               tg, dcnt, mid_list, long_list, stride, counters);
        PDP_TRY(hipGetLastError());
        // fixed grids; work-groups past the queued genes exit at once
        const dim3 mid_groups(std::min(tg, 2048u)), rest_groups(std::min(tg, 768u));
        if (narrow) {
            hipLaunchKernelGGL(k_mv_mid<true>, mid_groups, dim3(kMvThreads), 0, s, table, dcnt, mid_list, counters);
            PDP_TRY(hipGetLastError());
            hipLaunchKernelGGL(k_mv_rest<true>, rest_groups, dim3(kMvThreads), 0, s, table, dcnt, mid_list, stride,
                               long_list, counters);
        } else {
            hipLaunchKernelGGL(k_mv_mid<false>, mid_groups, dim3(kMvThreads), 0, s, table, dcnt, mid_list, counters);
            PDP_TRY(hipGetLastError());
            hipLaunchKernelGGL(k_mv_rest<false>, rest_groups, dim3(kMvThreads), 0, s, table, dcnt, mid_list, stride,
                               long_list, counters);
        }
        PDP_TRY(hipGetLastError());
    }
    PDP_TRY(launch_scan(dcnt, dcnt, tg, partials, s));  // in place: dcnt becomes the global offsets
    if (tg > 0) {
        if (narrow_rec)
            hipLaunchKernelGGL((k_mv_compact<true, true>), dim3(tg), dim3(kWave), 0, s, table, n, dcnt, ent_gene, ent_rec);
        else if (narrow)
            hipLaunchKernelGGL((k_mv_compact<true, false>), dim3(tg), dim3(kWave), 0, s, table, n, dcnt, ent_gene, ent_rec);
        else
            hipLaunchKernelGGL((k_mv_compact<false, false>), dim3(tg), dim3(kWave), 0, s, table, n, dcnt, ent_gene, ent_rec);
        PDP_TRY(hipGetLastError());
    }
    const bool few_bins = total_bins <= 8192;  // their scan by one work-group costs less than a launch
    if (narrow_rec)
        hipLaunchKernelGGL(k_ix_hist<true>, dim3(total_blocks), dim3(256), hist_lds, s, table, n,
                           dcnt, ent_rec, bintot, total_bins, few_bins ? binoff : nullptr, counters + 4);
    else
        hipLaunchKernelGGL(k_ix_hist<false>, dim3(total_blocks), dim3(256), hist_lds, s, table, n,
                           dcnt, ent_rec, bintot, total_bins, few_bins ? binoff : nullptr, counters + 4);
    PDP_TRY(hipGetLastError());
    if (!few_bins) PDP_TRY(launch_scan(bintot, binoff, total_bins, partials, s));  // every bin's range
    auto place = [&](auto kernel, uint32_t lds) {
        hipLaunchKernelGGL(kernel, dim3(total_blocks), dim3(kIxPlaceThreads), lds, s, table, n, dcnt, binoff, bintot,
                           ent_gene, ent_rec);
    };
    constexpr uint32_t kPer = kIxBlock / kIxPlaceThreads, kPerSmall = kIxBlockSmall / kIxPlaceThreads;
    const uint32_t stage_lds = 4 * ((max_nh + 1) & ~1u) + 8 * kIxBlock;
    if (narrow_rec) {
        if (small) {
            place(k_ix_place<uint2, kPerSmall, false>, hist_lds);
        } else if (stage_lds <= kMaxTileLds) {
            // the limit, not this build's size: another thread may be building with more bins
            PDP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(k_ix_place<uint2, kPer, true>),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(kMaxTileLds)));
            place(k_ix_place<uint2, kPer, true>, stage_lds);
        } else {
            place(k_ix_place<uint2, kPer, false>, hist_lds);
        }
    } else {
        if (small) place(k_ix_place<uint4, kPerSmall, false>, hist_lds);
        else place(k_ix_place<uint4, kPer, false>, hist_lds);
    }
    PDP_TRY(hipGetLastError());
    if (narrow_rec)
        hipLaunchKernelGGL(k_ix_sort_bin<uint2>, dim3(total_bins), dim3(BinSort<uint2>::kThreads), 0, s, table, n, binoff);
    else
        hipLaunchKernelGGL(k_ix_sort_bin<uint4>, dim3(total_bins), dim3(BinSort<uint4>::kThreads), 0, s, table, n, binoff);
    PDP_TRY(hipGetLastError());
    return hipSuccess;
}

}  // namespace pdp
