// Flat walk over staged runs of B entries (Thread-Flat-Parallel, Partitioning
// Schemes subsection): the products of a chunk of A entries numbered
// consecutively, neighbouring lanes on neighbouring products, so a run's loads
// coalesce and no lane idles past the end of a run.
#pragma once

#include "spg_internal.hpp"

namespace spg {

// The staging scan adds (run length) + (FLAT_ONE if the run is nonempty):
// products below the shift, the nonempty run's slot above it, so empty runs
// are not staged and run starts are distinct.
constexpr int FLAT_SHIFT = 48;
constexpr long long FLAT_ONE = 1ll << FLAT_SHIFT, FLAT_LEN = FLAT_ONE - 1;

// Products numbered in 32 bits: a chunk of `lanes` A entries forms at most
// nnz(B) products per entry (fewer in all unless A repeats a column), and a walk
// in rounds of `round` products steps past the last of them.
constexpr bool flat_32bit(int64_t nnzb, int lanes, int round) {
    return nnzb <= (INT32_MAX - round) / lanes;
}
static_assert(flat_32bit(33554423, 64, 512) && !flat_32bit(33554424, 64, 512), "last product number plus a round");
static_assert(flat_32bit(4194295, 512, 4096) && !flat_32bit(4194303, 512, 4096), "fits itself, its last round does not");

// k[u] = base + the bits of the window's mask (wb: 2 U words) below product
// u * 64 + lane: two counting instructions on masks that every lane shares.
template <int U>
__device__ __forceinline__ void flat_count(const uint32_t *wb, int base, int (&k)[U]) {
    const int l = lane_id();
    const uint2 m = l < U ? *(const uint2 *)&wb[2 * l] : make_uint2(0u, 0u);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint32_t lo = __builtin_amdgcn_readlane((int)m.x, u), hi = __builtin_amdgcn_readlane((int)m.y, u);
        k[u] = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, base));
        base += __builtin_popcount(lo) + __builtin_popcount(hi);
    }
}

// The run of every product of a wavefront's window [F, F + 64 U): runs have
// inclusive prefix ends off[0 .. cn) (increasing), wb is the wavefront's LDS
// scratch (2 U words), kc a run not behind the one that holds F.  Each run
// that starts inside the window sets the bit before its first product, and a
// product's run is the number of bits below it.  (Run numbers written at the
// starts and filled forward by a max-scan took nine per 64 products, and U LDS
// reads: R-MAT scale 17, both phases, 19.2 -> 18.8 ms, batch of 48 new values
// 2.80 -> 2.75, batch of 48 in full (column buckets) 9.90 -> 9.43 ms.)
// IX: a type that holds the chunk's product count.  Returns the first run of
// the window; k[u] is the run of product F + u * 64 + lane, relative to it
// (products past the chunk get its last run).
template <int U, typename IX>
__device__ __forceinline__ int flat_window(const IX *off, int cn, IX F, IX tot, int kc, uint32_t *wb, int (&k)[U]) {
    static_assert(2 * U <= WAVE, "a lane clears one word");
    const int l = lane_id();
    int klo = kc;
    if (off[klo] <= F) {
        int lo = klo + 1, hi = cn - 1;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (off[mid] > F) hi = mid;
            else lo = mid + 1;
        }
        klo = lo;
    }
    if (l < 2 * U) wb[l] = 0u;
    wave_lds_sync();
    const IX Fe = min(F + (IX)(U * WAVE), tot);
    for (int r = klo + 1 + l; r < cn; r += WAVE) {
        const IX st = off[r - 1];  // run r's first product, past F: run klo holds F
        if (st >= Fe) break;       // starts increase with r
        const int p = (int)(st - F) - 1;
        atomicOr(&wb[p >> 5], 1u << (p & 31));
    }
    wave_lds_sync();
    flat_count<U>(wb, 0, k);
    return klo;
}

}  // namespace spg
