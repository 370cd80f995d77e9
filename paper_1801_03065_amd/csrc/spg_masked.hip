// Masked product C = (A * B) on the pattern of a mask M, and its structural
// form (path counts): the graph-analytics use of SpGEMM the paper names in
// its Background section (triangle counting works on the structure of
// L * L restricted to L, Compression subsection).  No symbolic phase is
// needed: C's structure is M's.
//
// M's row goes into a linear-probing table (column -> position in M's row, at
// most 50% occupancy) next to a row of FP64 accumulators (FP32 inputs
// accumulate in FP64: the products of two FP32 numbers are exact there).  A
// product whose column is in the table is added at its position.  Products are
// walked flat, MK_U column loads in flight per lane, or, where rows have few of
// them, by groups of lanes per B row (mask_group).
//
// A row takes one wavefront, or a 512-lane workgroup (table in LDS; for mask
// rows beyond MG_MAX entries in a slice of an HBM arena behind an LDS bit
// filter: a column whose bit is clear is not in the row, so most products never
// touch the arena).  k_mask_class lists the rows (MaskList), mask_plan puts the
// lists into launches.  Workgroups take their rows from a queue, the longest
// first: the work per row spans four decades, and the few longest rows would leave
// most of the chip idle in a launch of their own.
//
// Bound by the latency of a product's column load and table read, so by
// products in flight: no unit is busy.  Triangles of an R-MAT graph, scale
// 18, 2.6M edges, 5.2e8 products: 1.86 ms a call, 0.28 products a ps; with lane
// groups for every row, one load in flight and one wavefront for any row of up to
// 512 mask entries it took 22 ms (a group of 16 lanes waited for the longest of
// four B rows, and one wavefront held rows of 1e6 products).
#include "spg_accum.hpp"
#include "spg_flat.hpp"
#include "spg_internal.hpp"

namespace spg {

namespace {

constexpr int MK_CB = 1024;  // classification
// Mask entries: a wavefront's row up to MW_MAX, or MW_LONG in launches of their own
// (the launch's LDS goes by its longest mask row); a workgroup's in LDS up to
// MG_MAX.  100k rows of 300 entries and 25 products: 306 us a call, as workgroups 1246.
constexpr int MW_MAX = 256, MW_LONG = 512, MG_MAX = 2048;
// Multiplications: up to MK_LIGHT a wavefront, beyond MK_F a workgroup.  Between them
// a workgroup where the product has up to MK_MID_WG such rows, a wavefront beyond:
// rows of 200 mask entries and 4000 multiplications 500 at a time 74 us as
// workgroups, 131 as wavefronts, 4000 146 and 169, 8000 223 and 205, 12000 301 and
// 236 (of 7500: 8000 333 and 329; of 2400: 4000 141 and 130).
constexpr int MK_LIGHT = 2048, MK_F = 8192, MK_MID_WG = 8192;
constexpr int MK_JOIN = 16384;   // rows up to which both lengths of wavefront rows share a launch
constexpr int MK_WG = 512;   // lanes of a workgroup row
constexpr int MK_U = 8;      // products per lane and round
constexpr int MK_FEWP = 64;  // a wavefront's chunk of up to as many products takes one round of one per lane
constexpr int MK_GROUP = 4, MK_TURNS = 4;  // (see mask_group)
static_assert(MK_GROUP <= MK_TURNS, "64 staged B rows in one round of turns");
constexpr int MK_FLG = 17, MK_FBITS = 1 << MK_FLG;  // bits of the filter of HBM rows

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

// Element i of an array that this kernel does not write, i the same in all lanes:
// a scalar load (a vector load of one address in 64 lanes takes the data unit as
// long as one of 64 addresses).
template <typename T>
__device__ __forceinline__ T mk_uniform(const T *p, int64_t i) {
    typedef const __attribute__((address_space(4))) T const_t;
    return ((const_t *)(uintptr_t)p)[i];
}
// Where a row's mask entries and A entries lie.
struct MkRow {
    int64_t mb, me, ab, ae;
};
template <typename VT>
__device__ __forceinline__ MkRow mk_row(const MaskArgs<VT> &a, int i) {
    if (i < 0) return MkRow{};
    return MkRow{mk_uniform(a.mrp, i), mk_uniform(a.mrp, i + 1), mk_uniform(a.arp, i), mk_uniform(a.arp, i + 1)};
}

// NW wavefronts per mask row.  lg, mmax: LDS table size (log2) and longest
// mask row held there; BIG: the first a.nrows3 rows are longer,
// their table is keys[cap] | posv[cap] | acc[cap / 2] in an arena slice (a.arena_slices of them); queue: row counter (NW > 1).
// WALK: products walked flat, or 2^a.lg_gs lanes per B row, none of which is longer
// (NW == 1; see mask_group): no scan and no search for a product's run, but lanes
// idle past a B row's end.
template <typename VT, typename IX, int NW, bool BIG, int WALK>
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
    const int64_t nrows = a.end[3];
    // Wavefront rows: a workgroup's rows are gridDim.x apart, so every die has its
    // share of each list (the lists differ in work per row: with an eighth of all
    // lists joined per die, triangles at scale 18 took 12% longer).  Groups: a
    // die's workgroups on rows next to each other, whose B rows its L2 then holds.
    int64_t r = WALK != MK_FLAT ? (int64_t)(blockIdx.x % XCDS) * (gridDim.x / XCDS) + blockIdx.x / XCDS : blockIdx.x;
    for (;;) {
        if (NW > 1) {
            if (t == 0) red[NW] = atomicAdd(queue, 1);
            __syncthreads();
            r = uni64(red[NW]);
        }
        if (r >= nrows) break;  // (a workgroup leaves once the queue's counter has passed the rows)
        const int q = (r >= a.end[0]) + (r >= a.end[1]) + (r >= a.end[2]);
        const int64_t r3 = r;
        const MkRow row = mk_row(a, mk_uniform(a.rows[q], r - (q ? a.end[q - 1] : 0)));
        if (NW == 1) r += gridDim.x;
        const bool big = BIG && r3 < a.nrows3;
        const int64_t mb = row.mb, ab = row.ab, ae = row.ae;
        const int ml = (int)(row.me - mb);
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
            long long inc, all;
            const int staged = (int)min((int64_t)WG, ae - c0);
            const bool grp = WALK == MK_GROUPS || (WALK == MK_EITHER && staged << a.lg_gs <= MK_TURNS * WAVE);
            if (grp) {
                mk_sync<NW>();  // (as below)
                off[t] = (IX)len;  // (0 past the chunk)
                rel[t] = (IX)b0;
                sav[t] = av;
                inc = all = 0;
            } else if constexpr (NW == 1 && sizeof(IX) == 4) {  // lane moves of 32 bits, runs counted on a mask
                const unsigned long long runs = __ballot(len > 0);
                const int sum = wave_scan_dpp((int)len);
                inc = sum + (long long)(mbcnt(runs) + 1) * FLAT_ONE;
                all = __builtin_amdgcn_readlane(sum, WAVE - 1) + (long long)__popcll(runs) * FLAT_ONE;
                mk_sync<NW>();  // the previous chunk's staging is no longer read; the table is complete
            } else {
                inc = wave_incl_scan64(len + (len > 0 ? FLAT_ONE : 0));
                all = __shfl(inc, WAVE - 1);
                mk_sync<NW>();  // (as above)
            }
            if constexpr (NW > 1) {
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
            if (!grp && len > 0) {
                const int k = (int)(inc >> FLAT_SHIFT) - 1;
                const long long end = inc & FLAT_LEN;
                off[k] = (IX)end;
                rel[k] = (IX)(b0 - (end - len));
                sav[k] = av;
            }
            mk_sync<NW>();
            // ---- products, U per lane and round
            auto products = [&](auto per_lane, auto groups) {
                constexpr int U = decltype(per_lane)::value;
                constexpr bool G = decltype(groups)::value;
                // G: one round of U turns, in each a B row per 2^lg_gs lanes: this lane's is
                // u * ng + g, below WAVE (one turn where lg_gs is 0, up to two where it is 1)
                const int lgg = G ? a.lg_gs : 0, ng = WAVE >> lgg, g = l >> lgg, p = l & ((1 << lgg) - 1);
                const IX end = G ? IX(1) : tot;
                int kc = 0;
                for (IX F = G ? IX(0) : (IX)wv * (U * WAVE); F < end; F += (IX)U * WG) {
                    int k[U], c[U], kk[U], at[U];
                    IX e[U];
                    if constexpr (G) {
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            k[u] = u * ng + g;
                            const IX b = rel[k[u]], n = off[k[u]];  // (read by every lane: no branch per product)
                            e[u] = p < n ? b + p : -1;
                        }
                    } else {
                        kc = flat_window<U>(off, cn, F, tot, kc, wb, k);
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            const IX f = F + (u * WAVE + l);
                            k[u] += kc;
                            const IX b = rel[k[u]];  // (as above: k[u] is a run of the chunk)
                            e[u] = f < tot ? b + f : -1;
                        }
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) c[u] = mk_ld(a.bci, max(e[u], IX(0)));
                    if (big) {
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            const uint32_t hb = mk_hash(c[u], MK_FLG);
                            kk[u] = (int)((filt[hb >> 5] >> (hb & 31)) & 1u);
                        }
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            at[u] = -1;
                            if (e[u] >= 0 && kk[u]) {
                                const uint32_t s = mk_hash(c[u], lgr);
                                at[u] = mk_probe<true>(gkeys, mask, c[u], s, mk_key<true>(gkeys, s));
                                if (at[u] >= 0) at[u] = gpos[at[u]];
                            }
                        }
                    } else {
#pragma unroll
                        for (int u = 0; u < U; ++u) kk[u] = keys[mk_hash(c[u], lgr)];
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            at[u] = -1;
                            if (e[u] >= 0 && kk[u] != -1) at[u] = mk_probe<false>(keys, mask, c[u], mk_hash(c[u], lgr), kk[u]);
                            if (at[u] >= 0) at[u] = posv[at[u]];
                        }
                    }
                    VT bv[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) bv[u] = !a.structural && at[u] >= 0 ? mk_ld(a.bval, e[u]) : VT(0);
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        if (at[u] >= 0) {
                            const double x = a.structural ? 1.0 : (double)sav[k[u]] * (double)bv[u];
                            if (big) atomicAdd(&gacc[at[u]], x);
                            else atomicAdd(&acc[at[u]], x);
                        }
                }
            };
            constexpr auto flat = std::false_type{};
            constexpr auto groups = std::true_type{};
            if (grp) {
                const int turns = ((staged << a.lg_gs) + WAVE - 1) / WAVE;
                if (turns == 1) products(std::integral_constant<int, 1>{}, groups);
                else if (turns == 2) products(std::integral_constant<int, 2>{}, groups);
                else products(std::integral_constant<int, MK_TURNS>{}, groups);
            } else if (NW == 1 && tot <= MK_FEWP) {
                products(std::integral_constant<int, MK_FEWP / WAVE>{}, flat);
            } else {
                products(std::integral_constant<int, MK_U>{}, flat);
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

// The rows' lists, with the longest mask row per list (see MaskList); rows with
// an empty mask row or an empty A row need no kernel (their outputs are
// zero-filled).  `its * 16` rows per workgroup, a lane each; where A's row and the
// longest row of B leave open which side of MK_LIGHT or MK_F a row's
// multiplications are on, 16 lanes sum them, one row after the other.  Per
// workgroup one atomic per list for the base of its slice.
__global__ __launch_bounds__(MK_CB) void k_mask_class(int64_t m, int64_t n, const int64_t *arp, const int32_t *aci,
                                                      const int64_t *brp, const int64_t *mrp, const int *longest, int its,
                                                      int32_t *rows, int *cnt) {
    constexpr int NONE = ML_N;
    __shared__ int sc[ML_N], sb[ML_N], smx[ML_N], open_n;
    __shared__ uint16_t open_rows[MK_CB];
    __shared__ uint8_t list[MK_CB];
    const int t = threadIdx.x, q = t & 15, per = its * (MK_CB / 16);
    if (t < ML_N) {
        sc[t] = 0;
        smx[t] = 0;
    }
    if (t == 0) open_n = 0;
    __syncthreads();
    const int64_t r0 = (int64_t)blockIdx.x * per, i = r0 + t;
    int k = NONE, ml = 0;
    if (t < per && i < m) {
        const int64_t mlen = mrp[i + 1] - mrp[i], la = arp[i + 1] - arp[i];
        if (mlen > 0 && la > 0) {
            ml = (int)min(mlen, (int64_t)INT_MAX);
            if (mlen > MG_MAX) k = ML_HBM;
            else if (mlen > MW_LONG) k = ML_WG;
            else {
                k = mlen > MW_MAX ? ML_LONG : ML_SHORT;
                if (la * *longest > MK_LIGHT) open_rows[atomicAdd(&open_n, 1)] = (uint16_t)t;
            }
        }
    }
    list[t] = (uint8_t)k;
    __syncthreads();
    for (int o = t >> 4; o < open_n; o += MK_CB / 16) {
        const int lr = open_rows[o];
        const int64_t ab = arp[r0 + lr], ae = arp[r0 + lr + 1];
        long long f = 0;
        for (int64_t e0 = ab; e0 < ae && f <= MK_F; e0 += 128) {  // (f <= MK_F: per lane, ends early)
            int j[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int64_t e = e0 + 16 * u + q;
                j[u] = e < ae ? aci[e] : -1;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (j[u] >= 0 && j[u] < n) f += brp[j[u] + 1] - brp[j[u]];
        }
#pragma unroll
        for (int d = 8; d >= 1; d >>= 1) f += __shfl_xor(f, d, 16);
        if (q == 0) list[lr] = f > MK_F ? ML_WG : f > MK_LIGHT ? list[lr] + 1 : list[lr];
    }
    __syncthreads();
    k = list[t];
    int my = 0;
    for (unsigned long long left = __ballot(k < NONE); left;) {  // one list of the wavefront at a time
        const int kk = __builtin_amdgcn_readlane(k, __ffsll((long long)left) - 1);
        const unsigned long long in = __ballot(k == kk);
        left &= ~in;
        const int longest_ml = __builtin_amdgcn_readlane(wave_maxscan_dpp(k == kk ? ml : 0), WAVE - 1);
        int at = 0;
        if (lane_id() == 0) {
            at = atomicAdd(&sc[kk], __popcll(in));
            atomicMax(&smx[kk], longest_ml);
        }
        at = read_first(at);  // lane 0's: with all lanes active
        if (k == kk) my = at + mbcnt(in);
    }
    __syncthreads();
    if (t < ML_N) {
        sb[t] = sc[t] ? atomicAdd(&cnt[t], sc[t]) : 0;
        if (smx[t] > *(volatile int *)&cnt[ML_N + t]) atomicMax(&cnt[ML_N + t], smx[t]);
    }
    __syncthreads();
    if (k < NONE) rows[(int64_t)k * m + sb[k] + my] = (int32_t)i;
}

template <typename VT, typename IX, int NW, bool BIG, int WALK = MK_FLAT>
hipError_t mask_ix(const MaskArgs<VT> &a, int mmax, int *queue, const LaunchCfg &c) {
    int lg = 4;
    while ((1 << lg) < 2 * mmax) ++lg;
    const size_t lds = mk_layout(NW * WAVE, lg, mmax, BIG).total;
    const int64_t rows = a.end[3];
    int grid = BIG ? c.grid : resident_grid(k_mask<VT, IX, NW, BIG, WALK>, NW * WAVE, lds, c.cus);
    // The flat walk's scalar registers leave room for 7 wavefronts per SIMD where the
    // occupancy query says 8; the eighth would start when the others are through
    // (200k rows of 1000 products: 710 us, with seven 606).
    if (NW == 1 && WALK == MK_FLAT) grid = std::min(grid, 28 * c.cus / XCDS * XCDS);
    grid = (int)std::min<int64_t>(grid, std::max<int64_t>(XCDS, ((rows + XCDS - 1) / XCDS) * XCDS));
    hipLaunchKernelGGL((k_mask<VT, IX, NW, BIG, WALK>), dim3(grid), dim3(NW * WAVE), lds, c.stream, a, lg, mmax, queue);
    return hipGetLastError();
}

// 32-bit product numbers and B indices where a chunk of A entries cannot form
// 2^31 products (nor B's values span 2^32 bytes): a quarter fewer instructions
// per product than 64-bit ones (triangles at scale 18: 2.16 against 2.27 ms in the two launches).
template <typename VT, int NW, bool BIG, int WALK = MK_FLAT>
hipError_t mask_impl(const MaskArgs<VT> &a, int mmax, int *queue, const LaunchCfg &c) {
    if (flat_32bit(a.nnzb, NW * WAVE, MK_U * NW * WAVE)) return mask_ix<VT, int32_t, NW, BIG, WALK>(a, mmax, queue, c);
    return mask_ix<VT, int64_t, NW, BIG, WALK>(a, mmax, queue, c);
}

}  // namespace

hipError_t launch_mask_class(int64_t m, int64_t n, const int64_t *arp, const int32_t *aci, const int64_t *brp,
                             const int64_t *mrp, const int *longest, int32_t *rows, int *cnt, hipStream_t s) {
    if (m == 0) return hipSuccess;
    // Small products: fewer rows one after the other per 16 lanes (2048 rows in
    // 16 turns: 26 us); large ones: one atomic per 1024 rows.  (With workgroups of a
    // quarter the size, 10k rows took 10.6 instead of 5.0 us: atomics on one counter.)
    const int its = (int)std::min<int64_t>(16, 2 * (1 + m / 65536));
    const int per = its * (MK_CB / 16);
    hipLaunchKernelGGL(k_mask_class, dim3((unsigned)((m + per - 1) / per)), dim3(MK_CB), 0, s, m, n, arp, aci, brp,
                       mrp, longest, its, rows, cnt);
    return hipGetLastError();
}

// A group of lanes per B row for groups of up to MK_GROUP lanes, and for wider ones
// where every row's A entries take up to MK_TURNS turns of 64 lanes: 100k rows of 300
// entries, B rows of one 282 us against 333 walked flat, of three or four 414 against
// 515; 7-point stencil 100^3 on its own pattern (one turn) 467 against 615, 200k rows
// of 4 entries times B rows of up to 64 (four) 231 against 290.  With more turns, in
// several rounds, idle lanes and fewer loads in flight cost more than the scan and
// the search (20k rows of 20 such entries 132 against 119 us).  Where only some rows
// take more, 64 A entries at a time one or the other: the two walks in one kernel
// hold a third more registers (the stencil 585, the 200k rows 261 us).
MaskWalk mask_group(int longest_b, int longest_a, int64_t m, int64_t nnza) {
    if (longest_b == 0 || longest_b > WAVE) return {MK_FLAT, 0};  // (a group's idle lanes load B's first entry)
    int lg = 0;
    while ((1 << lg) < longest_b) ++lg;
    if ((1 << lg) <= MK_GROUP || (int64_t)longest_a << lg <= MK_TURNS * WAVE) return {MK_GROUPS, lg};
    return {nnza << lg <= MK_TURNS * WAVE * m ? MK_EITHER : MK_FLAT, lg};
}

MaskPlan mask_plan(const int *n) {
    MaskPlan p{};
    const int mid = n[ML_SHORT_MID] + n[ML_LONG_MID];
    const bool mid_wg = mid <= MK_MID_WG;
    auto add = [&](int *lists, int &count, int list) {
        if (n[list] > 0) lists[count++] = list;
    };
    for (int list : {(int)ML_HBM, (int)ML_WG}) add(p.wg, p.wgs, list);
    if (mid_wg)
        for (int list : {(int)ML_LONG_MID, (int)ML_SHORT_MID}) add(p.wg, p.wgs, list);
    const int longs = n[ML_LONG] + (mid_wg ? 0 : n[ML_LONG_MID]);
    const int w = longs + n[ML_SHORT] + (mid_wg ? 0 : n[ML_SHORT_MID]) > MK_JOIN ? 1 : 0;
    if (!mid_wg) add(p.wave[0], p.waves[0], ML_LONG_MID);
    add(p.wave[0], p.waves[0], ML_LONG);
    if (!mid_wg) add(p.wave[w], p.waves[w], ML_SHORT_MID);
    add(p.wave[w], p.waves[w], ML_SHORT);
    return p;
}

template <typename VT>
hipError_t launch_mask(const MaskArgs<VT> &a, int mmax, int *queue, const LaunchCfg &c) {
    if (!queue && a.walk == MK_GROUPS) return mask_impl<VT, 1, false, MK_GROUPS>(a, mmax, nullptr, c);
    if (!queue && a.walk == MK_EITHER) return mask_impl<VT, 1, false, MK_EITHER>(a, mmax, nullptr, c);
    if (!queue) return mask_impl<VT, 1, false>(a, mmax, nullptr, c);
    if (a.nrows3 == 0) return mask_impl<VT, MK_WG / WAVE, false>(a, mmax, queue, c);
    return mask_impl<VT, MK_WG / WAVE, true>(a, mmax, queue, c);
}
template hipError_t launch_mask<double>(const MaskArgs<double> &, int, int *, const LaunchCfg &);
template hipError_t launch_mask<float>(const MaskArgs<float> &, int, int *, const LaunchCfg &);

}  // namespace spg
