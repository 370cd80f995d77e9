// Flat walk over staged runs of B entries (Thread-Flat-Parallel, Partitioning
// Schemes subsection): the products of a chunk of A entries numbered
// consecutively, neighbouring lanes on neighbouring products, so a run's loads
// coalesce and no lane idles past the end of a run.
#pragma once

#include "spg_internal.hpp"

namespace spg {

// Inclusive max-scan over the 64 lanes (values >= 0) with DPP lane moves.
__device__ __forceinline__ int wave_maxscan(int v) {
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false));  // row_shr:1
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false));  // row_shr:2
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false));  // row_shr:4
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false));  // row_shr:8
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false));  // row_bcast:15
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false));  // row_bcast:31
    return v;
}

// The staging scan adds (run length) + (FLAT_ONE if the run is nonempty):
// products below the shift, the nonempty run's slot above it, so empty runs
// are not staged and run starts are distinct.
constexpr int FLAT_SHIFT = 48;
constexpr long long FLAT_ONE = 1ll << FLAT_SHIFT, FLAT_LEN = FLAT_ONE - 1;

// The run of every product of a wavefront's window [F, F + 64 U): runs have
// inclusive prefix ends off[0 .. cn) (increasing), wi is the wavefront's LDS
// scratch (64 U entries), kc a run not behind the one that holds F.  Starts
// inside the window are marked in wi and filled forward by a max-scan.
// IX: a type that holds the chunk's product count.  Returns the first run of the window; k[u] is the run of product F + u * 64 +
// lane, relative to it (products past the chunk get its last run).
template <int U, typename IX>
__device__ __forceinline__ int flat_window(const IX *off, int cn, IX F, IX tot, int kc, uint16_t *wi, int (&k)[U]) {
    static_assert(U == 2 || U == 4 || U % 8 == 0, "a lane clears its entries with 4-, 8- or 16-byte stores");
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
    if constexpr (U == 2) {
        ((uint32_t *)wi)[l] = 0u;
    } else if constexpr (U == 4) {
        ((uint2 *)wi)[l] = make_uint2(0u, 0u);
    } else {
#pragma unroll
        for (int u = 0; u < U / 8; ++u) *(uint4 *)&wi[(u * WAVE + l) * 8] = make_uint4(0u, 0u, 0u, 0u);
    }
    wave_lds_sync();
    const IX Fe = min(F + (IX)(U * WAVE), tot);
    for (int r = klo + 1 + l; r < cn; r += WAVE) {
        const IX st = off[r - 1];  // run r's first product
        if (st >= Fe) break;       // starts increase with r
        wi[st - F] = (uint16_t)(r - klo);
    }
    wave_lds_sync();
#pragma unroll
    for (int u = 0; u < U; ++u) k[u] = wi[u * WAVE + l];
    int carry = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        k[u] = max(wave_maxscan(k[u]), carry);
        carry = __builtin_amdgcn_readlane(k[u], WAVE - 1);
    }
    return klo;
}

}  // namespace spg
