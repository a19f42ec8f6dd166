// Device helpers shared by the kernels of the pair path (pairs.hip) and of the group path
// (group.hip): exact comparison of similarities, candidate filters, column maxima.
#pragma once

#include "common.hpp"
#include "internal.hpp"

namespace pdp {

// Work-groups of a launch go to the XCDs in turn (work-group b to XCD b mod 8); item b' below gives
// XCD x a contiguous run of items.  The plan orders items by leading-letter bucket range across
// tasks, so an XCD works on one stretch of every genome's index at a time and its L2 serves
// the same slices to all the genome pairs that read them.
constexpr uint32_t kXcds = 8;
__device__ __forceinline__ uint32_t xcd_item(uint32_t b, uint32_t n) {
    const uint32_t q = n / kXcds, r = n % kXcds, x = b % kXcds;
    return x * q + min(x, r) + b / kXcds;  // a bijection of [0, n)
}

__device__ __forceinline__ bool j_greater(uint32_t m1, uint32_t d1, uint32_t m2, uint32_t d2) {
    return static_cast<uint64_t>(m1) * d2 > static_cast<uint64_t>(m2) * d1;
}
__device__ __forceinline__ bool j_equal(uint32_t m1, uint32_t d1, uint32_t m2, uint32_t d2) {
    return static_cast<uint64_t>(m1) * d2 == static_cast<uint64_t>(m2) * d1;
}

__device__ __forceinline__ uint32_t rec_min(uint32_t y) { return min(y & 0xFFFFu, y >> 16); }

// Candidate filters on one (row, column) pair: nr / nc windows of the two genes (their
// lengths are windows + k - 1: a pair with a shared k-mer has windows on both sides),
// sr / sc the occurrences of the shared k-mers in the row / column gene.  Eq.
// length_threshold: each length at least theta times the other; Eq. directional_jaccard:
// sr / nr and sc / nc at least tau.  Exact 64-bit products; a zero denominator is "off".
struct CandFilter {
    uint32_t k, theta_n, theta_d, tau_n, tau_d;
};
__device__ __forceinline__ bool candidate(const CandFilter &T, uint32_t nr, uint32_t nc, uint32_t sr, uint32_t sc) {
    if (T.theta_d) {
        const uint64_t lr = nr + T.k - 1, lc = nc + T.k - 1;
        if (lr * T.theta_d < uint64_t(T.theta_n) * lc || lc * T.theta_d < uint64_t(T.theta_n) * lr) return false;
    }
    if (T.tau_d) {
        if (uint64_t(sr) * T.tau_d < uint64_t(T.tau_n) * nr || uint64_t(sc) * T.tau_d < uint64_t(T.tau_n) * nc)
            return false;
    }
    return true;
}
__device__ __forceinline__ bool candidate(const DevTask &T, uint32_t nr, uint32_t nc, uint32_t sr, uint32_t sc) {
    return candidate(CandFilter{T.a.k, T.theta_n, T.theta_d, T.tau_n, T.tau_d}, nr, nc, sr, sc);
}

// Column maxima: the scratch of the tasks with kTaskColmax.
struct ColWs {
    unsigned long long *key;  // per best-hit row (a BA row): the running maximum key of its column
    uint4 *cands;             // pairs that reached their column's running maximum: (BA row, a, m, d)
    uint32_t *count;
    uint64_t cap;
};

// Key of J = m/d that orders values exactly: the bits of the correctly rounded double m / d.
// Distinct values differ by at least 1/(d1 d2) > 2^-34 (d < 2^17), far more than the rounding
// error (2^-53 relative, values at most 1), so their quotients keep their order; equal values
// round alike; positive doubles order as their bit patterns.  (An integer key floor(m 2^42 / d)
// orders them too, but its 64-bit division is a long instruction sequence per pair.)
__device__ __forceinline__ unsigned long long colmax_key(uint32_t m, uint32_t d) {
    return static_cast<unsigned long long>(__double_as_longlong(static_cast<double>(m) / static_cast<double>(d)));
}

// Raises the column's running maximum by the pair's key; true when the pair is at or above
// the maximum so far (the final maximum is never below it, so no final best hit is missed).
__device__ __forceinline__ bool colmax_raise(unsigned long long *key, uint32_t ba_row, uint32_t m, uint32_t d) {
    const unsigned long long k = colmax_key(m, d);
    return k >= atomicMax(&key[ba_row], k);
}

// The rows that get their hits from column maxima.
struct ColRows {
    uint32_t *bh_ptr;
    uint4 *slab;
    uint32_t *cursor;  // per row with more than kSlab hits: hits placed so far
    uint32_t *big;     // those rows
    uint32_t *n_big;
};

// Counts a hit (column, m, d) of a row, the first kSlab of them into its slab.
__device__ __forceinline__ void colmax_count(const ColRows &R, uint32_t row, uint32_t col, uint32_t m, uint32_t d) {
    const uint32_t t = atomicAdd(&R.bh_ptr[row], 1u);
    if (t < kSlab) {
        R.slab[static_cast<uint64_t>(row) * kSlab + t] = make_uint4(col, m, d, 0);
    } else if (t == kSlab) {  // one thread per row: the row is listed, its cursor cleared
        R.cursor[row] = 0;
        R.big[atomicAdd(R.n_big, 1u)] = row;
    }
}

// The best-hit output, after bh_ptr became row pointers.
struct ColCsr {
    const uint32_t *bh_ptr;
    uint32_t *col, *num, *den;
    uint64_t cap;
    uint32_t *cursor;
};

// Puts a hit of a row with more than kSlab of them into the output, in any order.
__device__ __forceinline__ void colmax_write(const ColCsr &C, uint32_t row, uint32_t col, uint32_t m, uint32_t d) {
    const uint32_t p = C.bh_ptr[row];
    if (C.bh_ptr[row + 1] - p <= kSlab) return;
    const uint64_t pos = uint64_t(p) + atomicAdd(&C.cursor[row], 1u);
    if (pos < C.cap) {
        C.col[pos] = col;
        C.num[pos] = m;
        C.den[pos] = d;
    }
}

}  // namespace pdp
