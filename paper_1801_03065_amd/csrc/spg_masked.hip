// Masked product C = (A * B) on the pattern of a mask M, and its structural
// form (path counts): the graph-analytics use of SpGEMM the paper names in
// its Background section (triangle counting works on the structure of
// L * L restricted to L, Compression subsection).  No symbolic phase is
// needed: C's structure is M's.
//
// M's row goes into a linear-probing table (column -> position in M's row, at
// most 50% occupancy) next to a row of FP64 accumulators (FP32 inputs
// accumulate in FP64: the products of two FP32 numbers are exact there).  The
// row's products are walked flat, MK_U column loads in flight per lane; one
// whose column is in the table is added at its position.
//
// Rows fall into three kinds (k_mask_class):
//   1. up to MW_MAX mask entries and MK_F multiplications (MK_F_FEW in products
//      of up to MK_FEW rows): one wavefront;
//   2. up to MG_MAX mask entries: one 512-lane workgroup, table in LDS;
//   3. longer mask rows: one 512-lane workgroup, table in a slice of an HBM
//      arena behind an LDS bit filter (a column whose bit is clear is not in
//      the row: most products never touch the arena).
// Kinds 3 and 2 share a launch and take rows from a queue, in that order: their
// work per row spans four decades, and the few longest rows would leave most
// of the chip idle in a launch of their own.
//
// Bound by the latency of a product's column load and table read, so by
// products in flight: no unit is busy (VALU 31 to 36%, LDS 12 to 17, data unit 28
// to 33; 50 to 61% of the wave cycles wait).  Triangles of an R-MAT graph, scale
// 18, 2.6M edges, 5.2e8 products: 2.0 ms in the two launches, 0.26 products a ps; with lane groups per B row, one load
// in flight and one wavefront for any row of up to 512 mask entries it took 22
// ms (a group of 16 lanes waited for the longest of four B rows, and one
// wavefront held rows of 1e6 products).
#include "spg_accum.hpp"
#include "spg_flat.hpp"
#include "spg_internal.hpp"

namespace spg {

namespace {

constexpr int MK_CB = 256;   // classification
constexpr int MK_FEW = 32768, MK_F_FEW = 2048;  // (see launch_mask_class)
constexpr int MK_WG = 512;   // lanes of a workgroup row
constexpr int MK_U = 8;      // products per lane and round
constexpr int MK_FLG = 17, MK_FBITS = 1 << MK_FLG;  // bits of the filter of kind 3

__device__ __forceinline__ uint32_t mk_hash(int c, uint32_t lg) {
    return ((uint32_t)c * 0x9E3779B1u) >> (32 - lg);
}

// LP insert of key c at position pos into keys/posv (size 2^lg); returns the slot.
template <typename P>
__device__ __forceinline__ int mk_insert(int *keys, P *posv, uint32_t lg, int c, int pos) {
    const uint32_t mask = (1u << lg) - 1u;
    uint32_t s = mk_hash(c, lg);
    for (;;) {
        const int prev = atomicCAS(&keys[s], -1, c);
        if (prev == -1 || prev == c) {
            posv[s] = (P)pos;
            return (int)s;
        }
        s = (s + 1) & mask;
    }
}

// Key in slot s.  HBM tables are read past the L1, which the inserts'
// compare-and-swaps do not go through.
template <bool HBM>
__device__ __forceinline__ int mk_key(const int *keys, uint32_t s) {
    return HBM ? __hip_atomic_load(&keys[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : keys[s];
}
// Slot of key c from its first probe (slot s, key k read there), or -1.
template <bool HBM>
__device__ __forceinline__ int mk_probe(const int *keys, uint32_t mask, int c, uint32_t s, int k) {
    while (k != c && k != -1) {
        s = (s + 1) & mask;
        k = mk_key<HBM>(keys, s);
    }
    return k == -1 ? -1 : (int)s;
}

// LDS of one workgroup of `wg` lanes; big: room for the bit filter.
struct MkLayout {
    size_t rel, off, av, red, wb, filt, keys, posv, acc, total;
};
__host__ __device__ inline MkLayout mk_layout(int wg, int lg, int mmax, bool big) {
    MkLayout L{};
    size_t o = 0;
    L.rel = o;  // per staged run: B entry of its first product, less that product's number
    o += 8 * (size_t)wg;
    L.off = o;  // inclusive prefix of the run lengths
    o += 8 * (size_t)wg;
    L.av = o;
    o += 8 * (size_t)wg;
    L.red = o;
    o += 8 * (size_t)(wg / WAVE + 2);
    L.wb = o;  // per wavefront: starts of the runs in its window (see flat_window)
    o += 8 * (size_t)MK_U * (wg / WAVE);
    o = align16(o);
    L.filt = o;
    if (big) o += MK_FBITS / 8;
    L.keys = o;
    o += 4 * ((size_t)1 << lg);
    L.posv = o;
    o += align16(2 * ((size_t)1 << lg));
    L.acc = o;
    o += 8 * (size_t)mmax;
    L.total = o;
    return L;
}

// B entry e: 32-bit byte offsets with a 32-bit index.
template <typename T>
__device__ __forceinline__ T mk_ld(const T *p, int32_t e) { return ld32(p, (uint32_t)e); }
template <typename T>
__device__ __forceinline__ T mk_ld(const T *p, int64_t e) { return p[e]; }

template <int NW>
__device__ __forceinline__ void mk_sync() {
    if constexpr (NW == 1) wave_lds_sync();
    else __syncthreads();
}

// NW wavefronts per mask row.  lg, mmax: LDS table size (log2) and longest
// mask row held there; BIG: the first a.nrows3 rows (list a.rows3) are longer,
// their table is keys[cap] | posv[cap] | acc[cap / 2] in an arena slice (a.arena_slices of them); queue: row counter (NW > 1).
template <typename VT, typename IX, int NW, bool BIG>
__global__ __launch_bounds__(NW *WAVE) void k_mask(MaskArgs<VT> a, int lg, int mmax, int *queue) {
    constexpr int WG = NW * WAVE;
    extern __shared__ __align__(16) unsigned char smem[];
    const MkLayout L = mk_layout(WG, lg, mmax, BIG);
    IX *rel = (IX *)(smem + L.rel);
    IX *off = (IX *)(smem + L.off);
    VT *sav = (VT *)(smem + L.av);
    long long *red = (long long *)(smem + L.red);
    const int t = threadIdx.x, l = lane_id(), wv = NW == 1 ? 0 : read_first(t / WAVE);
    uint32_t *wb = (uint32_t *)(smem + L.wb) + wv * (2 * MK_U);
    int *keys = (int *)(smem + L.keys);
    uint16_t *posv = (uint16_t *)(smem + L.posv);
    double *acc = (double *)(smem + L.acc);
    uint32_t *filt = (uint32_t *)(smem + L.filt);
    int *gkeys = nullptr, *gpos = nullptr;
    double *gacc = nullptr;
    if constexpr (BIG) {
        for (int s = t; s < MK_FBITS / 32; s += WG) filt[s] = 0;
    }
    for (int s = t; s < (1 << lg); s += WG) keys[s] = -1;
    for (int s = t; s < mmax; s += WG) acc[s] = 0.0;
    mk_sync<NW>();
    int badc = 0;
    const int64_t nrows = a.nrows + (BIG ? a.nrows3 : 0);
    const Slice sl = xcd_slice(0, nrows);
    int64_t r = sl.idx;
    for (;;) {
        if (NW == 1) {
            if (r >= sl.end) break;
        } else {
            if (t == 0) red[NW] = atomicAdd(queue, 1);
            __syncthreads();
            r = uni64(red[NW]);
            if (r >= nrows) break;  // every workgroup leaves here once the counter has passed the rows
        }
        const bool big = BIG && r < a.nrows3;
        const int64_t r3 = r;
        const int i = big ? a.rows3[r] : a.rows[r - (BIG ? a.nrows3 : 0)];
        r += sl.step;
        const int64_t mb = a.mrp[i];
        const int ml = (int)(a.mrp[i + 1] - mb);
        const int64_t ab = a.arp[i], ae = a.arp[i + 1];
        // this row's table: at most 25% occupied where the launch's size allows
        uint32_t lgr = min((uint32_t)lg, max(4u, 32u - (uint32_t)__clz(4 * ml - 1)));
        if (big) {
            // few such rows: one slice each; else one per workgroup
            const int64_t slice = a.nrows3 <= a.arena_slices ? r3 : (int64_t)blockIdx.x;
            unsigned char *base = (unsigned char *)a.arena + (size_t)slice * (size_t)a.arena_cap * 12;
            gkeys = (int *)base;
            gpos = (int *)(base + 4 * a.arena_cap);
            gacc = (double *)(base + 8 * a.arena_cap);
            lgr = 4;
            while (((int64_t)1 << lgr) < 2 * (int64_t)ml) ++lgr;
            if (((int64_t)1 << lgr) > a.arena_cap) {  // sized by the launch's longest mask row: cannot happen
                if (t == 0) atomicOr(a.bad, 2);
                __syncthreads();
                continue;
            }
            for (int64_t s = t; s < ((int64_t)1 << lgr); s += WG) gkeys[s] = -1;
            for (int64_t s = t; s < ml; s += WG) gacc[s] = 0.0;
            __threadfence();
            __syncthreads();
        }
        const uint32_t mask = (1u << lgr) - 1u;
        for (int e = t; e < ml; e += WG) {
            const int c = a.mci[mb + e];
            const bool okc = c >= 0 && c < a.k;
            badc |= !okc;
            if (!okc) continue;
            if (big) {
                mk_insert(gkeys, gpos, lgr, c, e);
                const uint32_t hb = mk_hash(c, MK_FLG);
                atomicOr(&filt[hb >> 5], 1u << (hb & 31));
            } else {
                mk_insert(keys, posv, lgr, c, e);
            }
        }
        if (big) __threadfence();
        for (int64_t c0 = ab; c0 < ae; c0 += WG) {
            // ---- stage the nonempty runs of up to WG A entries
            long long len = 0;
            int64_t b0 = 0;
            VT av = VT(0);
            if (c0 + t < ae) {
                const int j = a.aci[c0 + t];
                const bool okj = j >= 0 && j < a.n;
                badc |= !okj;
                if (okj) {
                    b0 = a.brp[j];
                    len = a.brp[j + 1] - b0;
                }
                if (a.aval) av = a.aval[c0 + t];
            }
            const long long v = len + (len > 0 ? FLAT_ONE : 0);
            long long inc = wave_incl_scan64(v), all;
            mk_sync<NW>();  // the previous chunk's staging is no longer read; the table is complete
            if (NW == 1) {
                all = __shfl(inc, WAVE - 1);
            } else {
                if (l == WAVE - 1) red[wv] = inc;
                __syncthreads();
                long long before = 0;
                all = 0;
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    before += w < wv ? red[w] : 0;
                    all += red[w];
                }
                inc += before;
            }
            const IX tot = (IX)(all & FLAT_LEN);
            const int cn = (int)(all >> FLAT_SHIFT);
            if (len > 0) {
                const int k = (int)(inc >> FLAT_SHIFT) - 1;
                const long long end = inc & FLAT_LEN;
                off[k] = (IX)end;
                rel[k] = (IX)(b0 - (end - len));
                sav[k] = av;
            }
            mk_sync<NW>();
            // ---- products, MK_U per lane and round
            int kc = 0;
            for (IX F = (IX)wv * (MK_U * WAVE); F < tot; F += (IX)MK_U * WG) {
                int k[MK_U], c[MK_U], kk[MK_U], at[MK_U];
                IX e[MK_U];
                kc = flat_window<MK_U>(off, cn, F, tot, kc, wb, k);
#pragma unroll
                for (int u = 0; u < MK_U; ++u) {
                    const IX f = F + (u * WAVE + l);
                    k[u] += kc;
                    e[u] = f < tot ? rel[k[u]] + f : -1;
                }
#pragma unroll
                for (int u = 0; u < MK_U; ++u) c[u] = mk_ld(a.bci, max(e[u], IX(0)));
                if (big) {
#pragma unroll
                    for (int u = 0; u < MK_U; ++u) {
                        const uint32_t hb = mk_hash(c[u], MK_FLG);
                        kk[u] = (int)((filt[hb >> 5] >> (hb & 31)) & 1u);
                    }
#pragma unroll
                    for (int u = 0; u < MK_U; ++u) {
                        at[u] = -1;
                        if (e[u] >= 0 && kk[u]) {
                            const uint32_t s = mk_hash(c[u], lgr);
                            at[u] = mk_probe<true>(gkeys, mask, c[u], s, mk_key<true>(gkeys, s));
                            if (at[u] >= 0) at[u] = gpos[at[u]];
                        }
                    }
                } else {
#pragma unroll
                    for (int u = 0; u < MK_U; ++u) kk[u] = keys[mk_hash(c[u], lgr)];
#pragma unroll
                    for (int u = 0; u < MK_U; ++u) {
                        at[u] = -1;
                        if (e[u] >= 0 && kk[u] != -1) at[u] = mk_probe<false>(keys, mask, c[u], mk_hash(c[u], lgr), kk[u]);
                        if (at[u] >= 0) at[u] = posv[at[u]];
                    }
                }
                VT bv[MK_U];
#pragma unroll
                for (int u = 0; u < MK_U; ++u) bv[u] = !a.structural && at[u] >= 0 ? mk_ld(a.bval, e[u]) : VT(0);
#pragma unroll
                for (int u = 0; u < MK_U; ++u)
                    if (at[u] >= 0) {
                        const double x = a.structural ? 1.0 : (double)sav[k[u]] * (double)bv[u];
                        if (big) atomicAdd(&gacc[at[u]], x);
                        else atomicAdd(&acc[at[u]], x);
                    }
            }
        }
        if (big) __threadfence();  // the HBM atomics complete before any lane reads an accumulator
        mk_sync<NW>();
        if (big) {
            for (int e = t; e < ml; e += WG)
                a.out[mb + e] = (VT)__hip_atomic_load(&gacc[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            for (int s = t; s < MK_FBITS / 32; s += WG) filt[s] = 0;
        } else {
            for (int e = t; e < ml; e += WG) {
                a.out[mb + e] = (VT)acc[e];
                acc[e] = 0.0;
            }
            for (int s = t; s < (1 << lgr); s += WG) keys[s] = -1;
        }
        mk_sync<NW>();
    }
    if (__ballot(badc) && l == 0) atomicOr(a.bad, 1);
}

// Row kinds, with the longest mask row per kind (see the file comment); rows
// with an empty mask row or an empty A row need no kernel (their outputs are
// zero-filled).  16 lanes sum a row's multiplications, `its` rows one after the
// other; per workgroup one atomic per kind for the base of its list slice.
__global__ __launch_bounds__(MK_CB) void k_mask_class(int64_t m, int64_t n, const int64_t *arp, const int32_t *aci,
                                                      const int64_t *brp, const int64_t *mrp, int its, int f_max, int32_t *rows,
                                                      int *cnt) {
    __shared__ int sc[3], sb[3], smx[3];
    __shared__ uint8_t kind[MK_CB];
    const int t = threadIdx.x, q = t & 15;
    if (t < 3) {
        sc[t] = 0;
        smx[t] = 0;
    }
    const int64_t r0 = (int64_t)blockIdx.x * (its * (MK_CB / 16));
    for (int it = 0; it < its; ++it) {
        const int lr = it * (MK_CB / 16) + (t >> 4);
        const int64_t i = r0 + lr;
        int k = 0;
        if (i < m) {
            const int64_t ml = mrp[i + 1] - mrp[i], ab = arp[i], ae = arp[i + 1];
            if (ml > 0 && ae > ab) {
                if (ml > MW_MAX) {
                    k = ml <= MG_MAX ? 2 : 3;
                } else {
                    long long f = 0;
                    for (int64_t e0 = ab; e0 < ae && f <= f_max; e0 += 64) {  // (f <= f_max: per lane, ends early)
                        int j[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const int64_t e = e0 + 16 * u + q;
                            j[u] = e < ae ? aci[e] : -1;
                        }
#pragma unroll
                        for (int u = 0; u < 4; ++u)
                            if (j[u] >= 0 && j[u] < n) f += brp[j[u] + 1] - brp[j[u]];
                    }
#pragma unroll
                    for (int d = 8; d >= 1; d >>= 1) f += __shfl_xor(f, d, 16);
                    k = f > f_max ? 2 : 1;
                }
            }
        }
        if (q == 0) kind[lr] = (uint8_t)k;
    }
    __syncthreads();
    const int64_t i = r0 + t;
    const int k = t < its * (MK_CB / 16) ? kind[t] : 0;
    int my = 0;
    if (k) {
        my = atomicAdd(&sc[k - 1], 1);
        atomicMax(&smx[k - 1], (int)min(mrp[i + 1] - mrp[i], (int64_t)INT_MAX));
    }
    __syncthreads();
    if (t < 3) {
        sb[t] = sc[t] ? atomicAdd(&cnt[t], sc[t]) : 0;
        if (smx[t]) atomicMax(&cnt[3 + t], smx[t]);
    }
    __syncthreads();
    if (k) rows[(int64_t)(k - 1) * m + sb[k - 1] + my] = (int32_t)i;
}

template <typename VT, typename IX, int NW, bool BIG>
hipError_t mask_ix(const MaskArgs<VT> &a, int mmax, int *queue, const LaunchCfg &c) {
    int lg = 4;
    while ((1 << lg) < 2 * mmax) ++lg;
    const size_t lds = mk_layout(NW * WAVE, lg, mmax, BIG).total;
    const int64_t rows = a.nrows + (BIG ? a.nrows3 : 0);
    int grid = BIG ? c.grid : resident_grid(k_mask<VT, IX, NW, BIG>, NW * WAVE, lds, c.cus);
    grid = (int)std::min<int64_t>(grid, std::max<int64_t>(XCDS, ((rows + XCDS - 1) / XCDS) * XCDS));
    hipLaunchKernelGGL((k_mask<VT, IX, NW, BIG>), dim3(grid), dim3(NW * WAVE), lds, c.stream, a, lg, mmax, queue);
    return hipGetLastError();
}

// 32-bit product numbers and B indices where a chunk of A entries cannot form
// 2^31 products (nor B's values span 2^32 bytes): a quarter fewer instructions
// per product than 64-bit ones (triangles at scale 18: 2.16 against 2.27 ms in the two launches).
template <typename VT, int NW, bool BIG>
hipError_t mask_impl(const MaskArgs<VT> &a, int mmax, int *queue, const LaunchCfg &c) {
    if (flat_32bit(a.nnzb, NW * WAVE, MK_U * NW * WAVE)) return mask_ix<VT, int32_t, NW, BIG>(a, mmax, queue, c);
    return mask_ix<VT, int64_t, NW, BIG>(a, mmax, queue, c);
}

}  // namespace

hipError_t launch_mask_class(int64_t m, int64_t n, const int64_t *arp, const int32_t *aci, const int64_t *brp,
                             const int64_t *mrp, int32_t *rows, int *cnt, hipStream_t s) {
    if (m == 0) return hipSuccess;
    // Small products: fewer rows one after the other per 16 lanes (2048 rows in
    // 16 turns: 26 us), and rows of MK_F_FEW multiplications already take a
    // workgroup, since the longest row alone decides (49 us).  A call at scale
    // 11: 82 us against 130; scale 12: 100 against 280 before the flat walk.
    // Large products: one atomic per 256 rows, and MK_F.
    const int its = (int)std::min<int64_t>(16, 1 + m / 16384);
    const int per = its * (MK_CB / 16);
    hipLaunchKernelGGL(k_mask_class, dim3((unsigned)((m + per - 1) / per)), dim3(MK_CB), 0, s, m, n, arp, aci, brp,
                       mrp, its, m <= MK_FEW ? MK_F_FEW : MK_F, rows, cnt);
    return hipGetLastError();
}

template <typename VT>
hipError_t launch_mask(const MaskArgs<VT> &a, int mmax, int *queue, const LaunchCfg &c) {
    if (!queue) return mask_impl<VT, 1, false>(a, mmax, nullptr, c);
    if (a.nrows3 == 0) return mask_impl<VT, MK_WG / WAVE, false>(a, mmax, queue, c);
    return mask_impl<VT, MK_WG / WAVE, true>(a, mmax, queue, c);
}
template hipError_t launch_mask<double>(const MaskArgs<double> &, int, int *, const LaunchCfg &);
template hipError_t launch_mask<float>(const MaskArgs<float> &, int, int *, const LaunchCfg &);

}  // namespace spg
