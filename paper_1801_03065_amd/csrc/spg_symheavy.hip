// Heavy rows, symbolic phase: the union of a row's column-set words in an LDS
// bit window over the row's whole column range (up to 2^20 columns), one
// workgroup per row.
//
// The row's words are walked flat over staged B rows, SH_U loads in flight per
// lane and neighbouring lanes on neighbouring words (spg_flat.hpp).  A word's
// bits are OR-ed only where they are not set yet: rows of power-law graphs meet
// their popular words from most B rows, and atomics on one LDS word serialise
// over the lanes while reads of it do not.  Then the words are counted, the
// row's segment list is cut (see k_num_sg), and where the numeric phase keeps
// heavy rows' structure the words themselves are stored.
//
// Bound by latency and by the LDS (counting, conflicting ORs).  R-MAT scale 17
// squared (1.5e9 compressed multiplications in 75k rows): 3.13 ms; with a
// binary search per word and a second OR into a summary word (which every 32nd
// word shares) it took 9.5 ms.
#include "spg_flat.hpp"
#include "spg_internal.hpp"

namespace spg {

namespace {

constexpr int SH_U = 8;  // words per lane and round

__host__ __device__ constexpr size_t align_up16(size_t x) { return (x + 15) & ~size_t(15); }

struct ShLayout {
    size_t bits, rel, off, wb, red, total;
};
__host__ __device__ inline ShLayout sh_layout(int nw_max, int wg, int ix_bytes) {
    ShLayout L{};
    size_t o = 0;
    L.bits = o;
    o += align_up16(4 * (size_t)nw_max);
    L.wb = o;
    o += 8 * (size_t)SH_U * (wg / WAVE);
    L.red = o;
    o += 8 * (size_t)(wg / WAVE + 2);
    L.rel = o;
    o += (size_t)ix_bytes * wg;
    L.off = o;
    o += 4 * (size_t)wg;
    L.total = o;
    return L;
}

// Block-wide exclusive scan; *total receives the sum (red: WG / WAVE longs).
template <int WG>
__device__ __forceinline__ long long sh_scan(long long v, long long *red, long long *total) {
    const int l = lane_id(), wv = threadIdx.x / WAVE;
    const long long inc = wave_incl_scan64(v);
    __syncthreads();
    if (l == WAVE - 1) red[wv] = inc;
    __syncthreads();
    long long off = 0, tot = 0;
#pragma unroll 4
    for (int u = 0; u < WG / WAVE; ++u) {
        const long long x = red[u];
        if (u < wv) off += x;
        tot += x;
    }
    *total = tot;
    return off + inc - v;
}

// COMP: compressed B.  IX: 32-bit B indices where byte offsets into the
// compressed B (or B's columns) fit 32 bits.
template <bool COMP, typename IX, int WG>
__global__ __launch_bounds__(WG) void k_sym_dg(SymArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    const ShLayout L = sh_layout(a.nw_max, WG, sizeof(IX));
    uint32_t *bits = (uint32_t *)(smem + L.bits);
    IX *rel = (IX *)(smem + L.rel);
    int *off = (int *)(smem + L.off);
    long long *red = (long long *)(smem + L.red);
    const int t = threadIdx.x, l = lane_id(), wv = read_first(t / WAVE);
    uint32_t *wb = (uint32_t *)(smem + L.wb) + wv * (2 * SH_U);
    for (int w = t; w < a.nw_max; w += WG) bits[w] = 0;
    int64_t lo, hi;
    rs_bounds(a.rs, lo, hi);
    int x = blockIdx.x % XCDS;
    const int64_t *srp = COMP ? a.bcrp : a.brp;
    for (;;) {
        __syncthreads();
        if (t == 0) {
            const int64_t q = xcd_grab(a.rs.queue, lo, hi, x);
            red[WG / WAVE] = q < 0 ? -1 : a.rs.rows[q];
        }
        __syncthreads();
        const int i = read_first((int)red[WG / WAVE]);  // scalar: so are the row's bounds
        if (i < 0) break;
        const int2 win = a.rwin[i];
        const int wlo = win.x, nw = win.y - win.x + 1;
        // a chunk's products stay below 2^31, the walk's last round included (a B
        // row holds up to 2^20 columns of a window, more only if it repeats them)
        const int64_t lim = (INT32_MAX - SH_U * WG) / WG;
        const int64_t ab = a.arp[i], ae = a.arp[i + 1];
        for (int64_t cb = ab; cb < ae; cb += WG) {
            int64_t b0 = 0, len = 0;
            if (cb + t < ae) {
                const int j = a.aci[cb + t];
                b0 = srp[j];
                len = min(srp[j + 1] - b0, lim);
            }
            long long all;
            const long long ex = sh_scan<WG>(len + (len > 0 ? FLAT_ONE : 0), red, &all);
            const int tot = read_first((int)(all & FLAT_LEN)), cn = read_first((int)(all >> FLAT_SHIFT));
            if (len > 0) {
                const int k = (int)(ex >> FLAT_SHIFT);
                const int before = (int)(ex & FLAT_LEN);
                off[k] = before + (int)len;
                rel[k] = (IX)(b0 - before);
            }
            __syncthreads();
            int kc = 0;
            for (int F = wv * (SH_U * WAVE); F < tot; F += SH_U * WG) {
                int k[SH_U];
                kc = flat_window<SH_U>(off, cn, F, tot, kc, wb, k);
                uint32_t d[SH_U], cs[SH_U];
                IX e[SH_U];
#pragma unroll
                for (int u = 0; u < SH_U; ++u) {
                    const int f = F + u * WAVE + l;
                    e[u] = f < tot ? rel[kc + k[u]] + f : rel[0];
                }
#pragma unroll
                for (int u = 0; u < SH_U; ++u) {
                    if constexpr (COMP) {
                        const uint2 v = sizeof(IX) == 4 ? ld32(a.bcw, (uint32_t)e[u]) : a.bcw[e[u]];
                        d[u] = v.x - (uint32_t)wlo;
                        cs[u] = v.y;
                    } else {
                        const int c = sizeof(IX) == 4 ? ld32(a.bci, (uint32_t)e[u]) : a.bci[e[u]];
                        d[u] = (uint32_t)((c >> 5) - wlo);
                        cs[u] = 1u << (c & 31);
                    }
                }
                // (lanes past the chunk repeat its first product)
                uint32_t cur[SH_U];
#pragma unroll
                for (int u = 0; u < SH_U; ++u) {
                    d[u] = min(d[u], (uint32_t)(nw - 1));
                    cur[u] = bits[d[u]];
                }
#pragma unroll
                for (int u = 0; u < SH_U; ++u)
                    if (cs[u] & ~cur[u]) atomicOr(&bits[d[u]], cs[u]);
            }
        }
        __syncthreads();
        // ---- count, cut and store the words, one aligned group of SG_NW at a
        // time: lane t has WPL consecutive words
        constexpr int WPL = SG_NW / WG;
        uint32_t *keep = a.sgb && a.sgb_len[i] > 0 ? a.sgb + a.sgb_off[i] : nullptr;
        const int cap = a.plan ? a.plan_len[i] : 0;
        uint2 *list = cap > 0 ? a.plan + a.plan_off[i] : nullptr;
        if (keep)
            for (int w = t; w < nw; w += WG) keep[w] = bits[w];
        long long run = 0, words = 0, cuts = 0;
        for (int g0 = 0; g0 < nw; g0 += SG_NW) {
            uint32_t m[WPL];
            const int w0 = g0 + t * WPL;
            long long c = 0;
#pragma unroll
            for (int u = 0; u < WPL; ++u) {
                m[u] = w0 + u < nw ? bits[w0 + u] : 0u;
                c += __popc(m[u]) + (m[u] ? 1ll << 32 : 0);
            }
            long long tot;
            const long long ex = sh_scan<WG>(c, red, &tot);
            if (list) {
                // a segment starts at the touched word that holds entry
                // q * SG_CUT for each q, and at the group's first touched word
                int p = (int)(run + (ex & 0xffffffffll)), nc = 0;
                unsigned cut = 0;
                bool first = (ex >> 32) == 0;
#pragma unroll
                for (int u = 0; u < WPL; ++u) {
                    const int cd = __popc(m[u]);
                    const int mult = ((p + SG_CUT - 1) / SG_CUT) * SG_CUT;  // first multiple of SG_CUT >= p
                    if (cd && (mult < p + cd || first)) {
                        cut |= 1u << u;
                        ++nc;
                    }
                    first = first && !cd;
                    p += cd;
                }
                long long ctot;
                long long idx = cuts + sh_scan<WG>(nc, red, &ctot);
                p = (int)(run + (ex & 0xffffffffll));
#pragma unroll
                for (int u = 0; u < WPL; ++u) {
                    if (cut & (1u << u)) {
                        if (idx + 2 < cap) list[1 + idx] = make_uint2((uint32_t)(w0 + u), (uint32_t)p);
                        ++idx;
                    }
                    p += __popc(m[u]);
                }
                cuts += ctot;
            }
            run += tot & 0xffffffffll;
            words += tot >> 32;
#pragma unroll
            for (int u = 0; u < WPL; ++u)
                if (w0 + u < nw) bits[w0 + u] = 0;
        }
        if (t == 0) {
            if (list) {
                // list[0] = (S, 0), list[1..S] = (first word, entries before it),
                // list[S + 1] = (window words, row size)
                if (cuts + 2 <= cap) {
                    list[0] = make_uint2((uint32_t)cuts, 0u);
                    list[1 + cuts] = make_uint2((uint32_t)nw, (uint32_t)run);
                } else {
                    atomicAdd(&a.st->overflow, 1);
                }
            }
            a.row_nnz[i] = (int32_t)run;
            a.row_words[i] = (int32_t)words;
        }
    }
}

template <bool COMP, typename IX, int WG>
hipError_t sym_dg_wg(const SymArgs &a, const LaunchCfg &c) {
    const size_t lds = sh_layout(a.nw_max, WG, sizeof(IX)).total;
    int grid = resident_grid(k_sym_dg<COMP, IX, WG>, WG, lds, c.cus);
    if (c.grid > 0) grid = std::max(XCDS, std::min(grid, c.grid) / XCDS * XCDS);
    hipLaunchKernelGGL((k_sym_dg<COMP, IX, WG>), dim3(grid), dim3(WG), lds, c.stream, a);
    return hipGetLastError();
}

// 512 lanes while the LDS window leaves room for several workgroups per CU (a
// row then has a workgroup of its size), 1024 beyond.
template <bool COMP, typename IX>
hipError_t sym_dg_ix(const SymArgs &a, const LaunchCfg &c) {
    if (a.nw_max <= 2 * SG_NW) return sym_dg_wg<COMP, IX, 512>(a, c);
    return sym_dg_wg<COMP, IX, 1024>(a, c);
}

}  // namespace

hipError_t launch_sym_dg(const SymArgs &a, const LaunchCfg &c) {
    if (a.bcrp) return a.b32 ? sym_dg_ix<true, int32_t>(a, c) : sym_dg_ix<true, int64_t>(a, c);
    return a.b32 ? sym_dg_ix<false, int32_t>(a, c) : sym_dg_ix<false, int64_t>(a, c);
}

}  // namespace spg
