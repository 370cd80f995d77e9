// Scattered rows in column buckets (numeric phase).
//
// A row of C whose products rarely meet (random or very sparse operands: at
// most two products per entry on average) needs its products sorted far more
// than it needs an accumulator.  The kernel sorts them by one counting pass:
//
//   1. every product (column, A value * B value) is loaded once into
//      registers, U per lane, neighbouring lanes on neighbouring products
//      (the owner of a product: run starts of the B rows marked in LDS, counted
//      on the marks), so no lane idles past the end of a B row;
//   2. the row's column window is cut into as many equal buckets as the
//      lanes hold products (a monotone map of the column); an LDS counter per
//      bucket gives every product its place in the bucket, a scan gives each
//      bucket its place in the row;
//   3. a product's place in the sorted row is its bucket's start plus the
//      products of the bucket that sort before it (about one other to look
//      at when columns are spread evenly);
//   4. products of one column are neighbours now: the first of them sums the
//      run and writes the entry; without repeats the row is written as it is.
//      (In the order of the bucket counter, which is free over the wavefronts of
//      a row: sums can differ in their last bits from run to run.)
//
// Rows with columns clustered inside the window (a bucket of more than BK_SPLIT
// products: power-law graphs) cut every bucket again in proportion to its
// products; the few that still have a bucket of more than BK_DEEP are sorted
// by a bitonic network instead of steps 2 and 3.
//
// Rows of up to 512 products take one wavefront, of up to 1024 and 2048 two
// and four (LDS and registers would leave one wavefront of 16 products per
// lane at 8 per CU: 12.5 ps a product against 9.3 with two).  LDS is 16 B per
// product (FP64), in launches of 64 * U * NW products, so short rows do not
// pay for the LDS of long ones.
//
// Measured on the batch of 48 random products (FP64, 24 B moved per product
// in and out): 8.1 to 10.0 ps a product over rows of 65 to 2048 products,
// 2.4 to 3.0 TB/s; bound by memory latency at 16 wavefronts per CU (registers).
// The kernels it replaces there: column hash with its bitonic sort 94 ps, word
// hash 58, segments 21 (29.3, 14.1 and 1.6 ms; the five launches here 5.0 ms).
#include "spg_accum.hpp"
#include "spg_flat.hpp"
#include "spg_internal.hpp"

namespace spg {

namespace {

constexpr int BK_SPLIT = 12;  // products of one bucket above which the buckets are cut again (even columns: 5 to 7)
constexpr int BK_DEEP = 24;   // and then above which the row is sorted by the network

struct RowDescB {
    int64_t ab, cb, ce;
    int na, wlo, nw;
};

__device__ __forceinline__ RowDescB row_desc_b(int i, const int64_t *arp, const int2 *rwin, const int64_t *coff) {
    RowDescB d;
    d.ab = arp[i];
    d.na = (int)min((int64_t)WAVE, arp[i + 1] - d.ab);
    d.cb = coff[i];
    d.ce = coff[i + 1];
    const int2 w = rwin[i];
    d.wlo = w.x;
    d.nw = w.y - w.x + 1;
    return d;
}

// Hand-over of LDS data between the lanes of the workgroup.  Both forms wait
// for LDS only, so loads for the next row stay in flight.
template <int NW>
__device__ __forceinline__ void bk_sync() {
    if constexpr (NW == 1) {
        wave_lds_sync();
    } else {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt = 0
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    }
}

// Marks in wb (2 U words, this wavefront's) the bit before the first product of
// each nonempty run (products [ex, ex + len)) that starts inside the
// wavefront's products after the first of them; returns the runs that start
// before, less the row's first.
template <int NW, int U>
__device__ __forceinline__ int bk_starts(uint32_t *wb, int len, int ex, int wv) {
    const int l = lane_id();
    if (l < 2 * U) wb[l] = 0u;
    wave_lds_sync();
    const int p = ex - 1 - wv * (WAVE * U);
    if (len > 0 && (unsigned)p < (unsigned)(WAVE * U)) atomicOr(&wb[p >> 5], 1u << (p & 31));
    return NW == 1 ? 0 : __popcll(__ballot(len > 0 && ex > 0 && p < 0));
}

// NW wavefronts per row, U products per lane.
template <typename VT, int ACC, int NW, int U>
__global__ __launch_bounds__(WAVE * NW) __attribute__((amdgpu_waves_per_eu(4))) void k_num_bk(NumArgs<VT> a) {
    using Term = BkTerm<VT, ACC>;
    using P = typename Term::term_t;
    constexpr int WG = WAVE * NW, CAP = WG * U;  // CAP: products of a row, and buckets
    __shared__ __align__(16) uint32_t cnt[CAP];  // bucket: count, then start | count << 16
    __shared__ __align__(16) int32_t key[CAP];   // columns in bucket order, then sorted
    __shared__ __align__(16) unsigned char val_raw[CAP * sizeof(P)];
    __shared__ int32_t st_rel[WAVE];             // per nonempty B row: its start - its first product
    __shared__ VT st_a[WAVE];
    __shared__ __align__(8) uint32_t starts[NW][2 * U];  // per wavefront: B row starts (see spg_flat.hpp)
    __shared__ int red[2 * NW + 2];
    P *val = (P *)val_raw;  // products in sorted order
    const int t = threadIdx.x, l = lane_id(), wv = NW == 1 ? 0 : read_first(t / WAVE);
    const int p0 = wv * (WAVE * U) + l;   // this lane's products: p0 + u * WAVE
#pragma unroll
    for (int u = 0; u < U; ++u) cnt[u * WG + t] = 0;
    int64_t lo, hi;
    rs_bounds(a.rs, lo, hi);
    const int64_t cbase = a.cbase_row >= 0 ? a.coff[a.cbase_row] : 0;
    const uint32_t elast = (uint32_t)(a.nnzb - 1);
    const Slice sl = xcd_slice(lo, hi);
    // Software pipeline across rows, as in the other wavefront kernels: the
    // next row's A entries (first level), then its B row extents (second
    // level), and the descriptor of the row after it load during this row.
    // Every wavefront of the row holds the A entries (one per lane).
    int64_t r = sl.idx;
    RowDescB dcur = r < sl.end ? row_desc_b(a.rs.rows[r], a.arp, a.rwin, a.coff) : RowDescB{};
    int64_t b0 = 0, b1 = 0;
    VT av = VT(0);
    if (r < sl.end && l < dcur.na) {
        const int j = a.aci[dcur.ab + l];
        av = a.aval[dcur.ab + l];
        b0 = a.brp[j];
        b1 = a.brp[j + 1];
    }
    RowDescB dn = r + sl.step < sl.end ? row_desc_b(a.rs.rows[r + sl.step], a.arp, a.rwin, a.coff) : RowDescB{};
    while (r < sl.end) {
        const RowDescB d = dcur;
        r += sl.step;
        const bool has_next = r < sl.end;
        // ---- products of the row: prefix of the B row lengths, owners
        const int len = l < d.na ? (int)(b1 - b0) : 0;
        const int inc = wave_scan_dpp(len), ex = inc - len;
        const int f = __builtin_amdgcn_readlane(inc, WAVE - 1);
        const int64_t n64 = d.ce - d.cb;
        const bool fits = f > 0 && f <= CAP && n64 <= f;  // else the structure changed behind the plan
        if ((NW == 1 || wv == 0) && len > 0) {
            const int run = mbcnt(__ballot(len > 0));
            st_rel[run] = (int32_t)b0 - ex;
            st_a[run] = av;
        }
        // runs that start before this wavefront's products; the others' starts
        const int base = bk_starts<NW, U>(starts[wv], len, ex, wv);
        if (NW > 1 && t < 2) red[2 * NW + t] = 0;
        // next row, first level
        const int nna = has_next ? dn.na : 0;
        int nj = 0;
        if (l < nna) {
            nj = a.aci[dn.ab + l];
            av = a.aval[dn.ab + l];
        }
        bk_sync<NW>();
        int col[U], k[U];
        VT bv[U];
        flat_count<U>(starts[wv], base, k);
        uint32_t e[U], kp[(U + 3) / 4] = {};  // kp: the runs (below 64) packed, four to a register
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int p = u * WAVE + p0;
            e[u] = p < f ? min((uint32_t)(st_rel[k[u]] + p), elast) : 0u;
            kp[u / 4] |= (uint32_t)k[u] << (8 * (u % 4));
        }
#pragma unroll
        for (int u = 0; u < U; ++u) col[u] = ld32(a.bci, e[u]);
#pragma unroll
        for (int u = 0; u < U; ++u) bv[u] = ld32(a.bval, e[u]);
        // next row, second level; the row after it: descriptor
        if (l < nna) {
            b0 = a.brp[nj];
            b1 = a.brp[nj + 1];
        }
        dcur = dn;
        if (r + sl.step < sl.end) dn = row_desc_b(a.rs.rows[r + sl.step], a.arp, a.rwin, a.coff);
        if (!fits) {  // the same in every wavefront of the row
            if (t == 0) atomicAdd(&a.st->mismatch, 1);
            bk_sync<NW>();
            continue;
        }
        const int n = (int)n64;

        // ---- buckets: monotone map of the window onto CAP buckets (the scale
        // is rounded down, so the window's last column stays below CAP)
        const int c0 = d.wlo << 5;
        const float w = 32.0f * (float)d.nw;
        const uint32_t scale = (uint32_t)fminf((float)CAP * 4294967296.0f * 0.999998f * __builtin_amdgcn_rcpf(w),
                                               4294967040.0f);
        uint32_t bs[U];  // bucket | place in it << 16
#pragma unroll
        for (int u = 0; u < U; ++u)
            bs[u] = min(__umulhi((uint32_t)(col[u] - c0), scale), (uint32_t)(CAP - 1));
        // Places in the buckets, then the buckets' starts (cnt: start | count
        // << 16); returns the largest bucket.
        auto count = [&]() -> int {
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (u * WAVE + p0 < f) bs[u] |= atomicAdd(&cnt[bs[u]], 1u) << 16;
            bk_sync<NW>();
            uint32_t cc[U];  // lane t scans buckets [t * U, (t + 1) * U)
            int sum = 0, mx = 0;
#pragma unroll
            for (int u = 0; u < U; ++u) cc[u] = cnt[t * U + u];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                sum += (int)cc[u];
                mx = max(mx, (int)cc[u]);
            }
            const int incs = wave_scan_dpp(sum);
            int run = incs - sum, dp = __builtin_amdgcn_readlane(wave_maxscan_dpp(mx), WAVE - 1);
            if (NW > 1) {
                if (l == WAVE - 1) {
                    red[wv] = incs;
                    red[NW + wv] = dp;
                }
                bk_sync<NW>();
#pragma unroll
                for (int v = 0; v < NW; ++v) {
                    run += v < wv ? red[v] : 0;
                    dp = max(dp, red[NW + v]);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                cnt[t * U + u] = (uint32_t)run | (cc[u] << 16);
                run += (int)cc[u];
            }
            bk_sync<NW>();
            return read_first(dp);
        };
        int deep = count();
        if (deep > BK_SPLIT) {
            // Columns clustered in the window: each bucket is cut again into
            // as many equal parts as it holds products.
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t xb = cnt[bs[u] & 0xFFFFu], part = (uint32_t)(col[u] - c0) * scale;  // place inside it
                bs[u] = min((xb & 0xFFFFu) + __umulhi(part, xb >> 16), (uint32_t)(CAP - 1));
            }
            bk_sync<NW>();
#pragma unroll
            for (int u = 0; u < U; ++u) cnt[u * WG + t] = 0;
            bk_sync<NW>();
            deep = count();
        }

        // ---- place of each product in the sorted row (left in bs)
        const bool net = deep > BK_DEEP;
        bool repeats = true;  // some column met twice
        if (!net) {
            uint32_t sc[U];  // bucket start | products << 16
#pragma unroll
            for (int u = 0; u < U; ++u) {
                sc[u] = cnt[bs[u] & 0xFFFFu];
                bs[u] >>= 16;
                if (u * WAVE + p0 >= f) sc[u] = 0;
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (u * WAVE + p0 < f) key[(sc[u] & 0xFFFFu) + bs[u]] = col[u];
            bk_sync<NW>();
            bool seen = false;
            int pos[U];
#pragma unroll
            for (int u = 0; u < U; ++u) pos[u] = (int)(sc[u] & 0xFFFFu);
            for (int j = 0; j < deep; ++j) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (j < (int)(sc[u] >> 16)) {
                        const int kj = key[(sc[u] & 0xFFFFu) + j];
                        const bool same = kj == col[u] && j < (int)bs[u];
                        seen |= same;
                        pos[u] += (kj < col[u] || same) ? 1 : 0;
                    }
                }
            }
            repeats = __ballot(seen) != 0;
            if (NW > 1 && repeats && l == 0) red[2 * NW] = 1;
            bk_sync<NW>();
            if (NW > 1) repeats = red[2 * NW] != 0;
#pragma unroll
            for (int u = 0; u < U; ++u) bs[u] = (uint32_t)pos[u];
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) bs[u] = (uint32_t)(u * WAVE + p0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (u * WAVE + p0 < f) {
                key[bs[u]] = col[u];
                val[bs[u]] = Term::term(st_a[(kp[u / 4] >> (8 * (u % 4))) & 0xFFu], bv[u]);
            }
        }
        if (net) {
            int np = WAVE;
            while (np < f) np <<= 1;
            for (int p = f + t; p < np; p += WG) key[p] = INT_MAX;
            bk_sync<NW>();
            for (int kk = 2; kk <= np; kk <<= 1)
                for (int j = kk >> 1; j > 0; j >>= 1) {
                    for (int p = t; p < (np >> 1); p += WG) {
                        const int i1 = ((p & ~(j - 1)) << 1) | (p & (j - 1)), i2 = i1 + j;
                        const bool up = (i1 & kk) == 0;
                        const int32_t k1 = key[i1], k2 = key[i2];
                        if ((k1 > k2) == up) {
                            key[i1] = k2;
                            key[i2] = k1;
                            const P v1 = val[i1];
                            val[i1] = val[i2];
                            val[i2] = v1;
                        }
                    }
                    bk_sync<NW>();
                }
        }
        bk_sync<NW>();

        // ---- write the row: each run of one column summed by its first product
        const int64_t ob = d.cb - cbase;
        if (!repeats && f == n) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int p = u * WAVE + p0;
                if (p < f) {
                    Term s;
                    s.add(val[p]);
                    store_c(&a.cci[ob + p], key[p]);
                    store_c(&a.cval[ob + p], s.fin());
                }
            }
        } else {
            unsigned long long head[U];
            int kc[U], total = 0, base = 0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int p = u * WAVE + p0;
                kc[u] = p < f ? key[p] : -1;
                head[u] = __ballot(p < f && (p == 0 || key[p - 1] != kc[u]));
                total += __popcll(head[u]);
            }
            if (NW > 1) {
                if (l == 0) red[wv] = total;
                bk_sync<NW>();
                total = 0;
#pragma unroll
                for (int v = 0; v < NW; ++v) {
                    base += v < wv ? red[v] : 0;
                    total += red[v];
                }
            }
            if (total != n) {
                if (t == 0) atomicAdd(&a.st->mismatch, 1);
            } else {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if ((head[u] >> l) & 1ull) {
                        int p = u * WAVE + p0;
                        Term s;
                        do s.add(val[p]);
                        while (++p < f && key[p] == kc[u]);
                        const int64_t o = ob + base + mbcnt(head[u]);
                        store_c(&a.cci[o], kc[u]);
                        store_c(&a.cval[o], s.fin());
                    }
                    base += __popcll(head[u]);
                }
            }
        }
        bk_sync<NW>();
#pragma unroll
        for (int u = 0; u < U; ++u) cnt[u * WG + t] = 0;
    }
}

// Symbolic phase of scattered rows: the same product walk over the columns
// alone, distinct columns counted by a linear-probing hash in LDS (two slots
// per product, so at most half full; all first probes of a lane in flight
// together).  Batch of 48 random products (6.1e8 products): 2.2 ms in the
// launches of 65 to 2048 products, against 5.8 ms for the bit window, which
// clears, ORs and counts 2048 words and their summary per row and holds a lane
// group of 32 per B row of 4 to 32 entries.  Random 1.5M rows: 144 us against
// 404 for the one-probe-at-a-time column hash.
template <int NW, int U>
__global__ __launch_bounds__(WAVE * NW) void k_sym_bk(SymArgs a) {
    constexpr int WG = WAVE * NW, CAP = WG * U, SLOTS = 2 * CAP;
    constexpr int LG = __builtin_ctz(SLOTS);
    __shared__ __align__(16) int32_t tab[SLOTS];
    __shared__ __align__(8) uint32_t starts[NW][2 * U];
    __shared__ int32_t st_rel[WAVE];
    __shared__ int red[NW];
    const int t = threadIdx.x, l = lane_id(), wv = NW == 1 ? 0 : read_first(t / WAVE);
    const int p0 = wv * (WAVE * U) + l;
#pragma unroll
    for (int u = 0; u < SLOTS / WG; ++u) tab[u * WG + t] = -1;
    int64_t lo, hi;
    rs_bounds(a.rs, lo, hi);
    const uint32_t elast = (uint32_t)(a.nnzb - 1);
    const Slice sl = xcd_slice(lo, hi);
    // software pipeline across rows: the next row's A entries, then their B
    // row extents, and the row after it's bounds load during this row
    auto bounds = [&](int64_t q, int &i, int64_t &ab, int &na) {
        i = -1;
        na = 0;
        if (q < sl.end) {
            i = a.rs.rows[q];
            ab = a.arp[i];
            na = (int)min((int64_t)WAVE, a.arp[i + 1] - ab);
        }
    };
    int64_t r = sl.idx, ab = 0, nab = 0, b0 = 0, b1 = 0;
    int i, na, ni, nna;
    bounds(r, i, ab, na);
    bounds(r + sl.step, ni, nab, nna);
    if (l < na) {
        const int j = a.aci[ab + l];
        b0 = a.brp[j];
        b1 = a.brp[j + 1];
    }
    while (r < sl.end) {
        const int row = i;
        r += sl.step;
        const int len = l < na ? (int)(b1 - b0) : 0;
        const int inc = wave_scan_dpp(len), ex = inc - len;
        const int f = min(__builtin_amdgcn_readlane(inc, WAVE - 1), CAP);
        if ((NW == 1 || wv == 0) && len > 0) st_rel[mbcnt(__ballot(len > 0))] = (int32_t)b0 - ex;
        const int base = bk_starts<NW, U>(starts[wv], len, ex, wv);
        int nj = 0;
        if (l < nna) nj = a.aci[nab + l];
        bk_sync<NW>();
        int col[U];
        flat_count<U>(starts[wv], base, col);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int p = u * WAVE + p0;
            col[u] = p < f ? (int)min((uint32_t)(st_rel[col[u]] + p), elast) : 0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) col[u] = ld32(a.bci, (uint32_t)col[u]);
        na = nna;
        if (l < nna) {
            b0 = a.brp[nj];
            b1 = a.brp[nj + 1];
        }
        i = ni;
        bounds(r + sl.step, ni, nab, nna);
        // ---- distinct columns
        uint32_t h[U];
        int old[U], fresh = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            h[u] = ((uint32_t)col[u] * 0x9E3779B1u) >> (32 - LG);
            old[u] = col[u];
            if (u * WAVE + p0 < f) old[u] = atomicCAS(&tab[h[u]], -1, col[u]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            while (old[u] != -1 && old[u] != col[u]) {
                h[u] = (h[u] + 1) & (SLOTS - 1);
                old[u] = atomicCAS(&tab[h[u]], -1, col[u]);
            }
            fresh += old[u] == -1;
        }
        int n = __builtin_amdgcn_readlane(wave_scan_dpp(fresh), WAVE - 1);
        if (NW > 1) {
            if (l == 0) red[wv] = n;
            bk_sync<NW>();
            n = 0;
#pragma unroll
            for (int v = 0; v < NW; ++v) n += red[v];
        }
        if (t == 0) {
            const int2 w = a.rwin[row];
            a.row_nnz[row] = n;
            a.row_words[row] = min(n, w.y - w.x + 1);  // a bound
        }
        bk_sync<NW>();
#pragma unroll
        for (int u = 0; u < SLOTS / WG; ++u) tab[u * WG + t] = -1;
    }
}

int grid_of(int resident, int64_t rows) {
    return (int)std::min<int64_t>(resident, std::max<int64_t>(XCDS, (rows + XCDS - 1) / XCDS * XCDS));
}

template <int NW, int U>
hipError_t sym_bk_u(const SymArgs &a, const LaunchCfg &c, int64_t rows) {
    const int grid = grid_of(resident_grid(k_sym_bk<NW, U>, WAVE * NW, 0, c.cus), rows);
    hipLaunchKernelGGL((k_sym_bk<NW, U>), dim3(grid), dim3(WAVE * NW), 0, c.stream, a);
    return hipGetLastError();
}

template <typename VT, int ACC, int NW, int U>
hipError_t num_bk_u(const NumArgs<VT> &a, const LaunchCfg &c, int64_t rows) {
    const int grid = grid_of(resident_grid(k_num_bk<VT, ACC, NW, U>, WAVE * NW, 0, c.cus), rows);
    hipLaunchKernelGGL((k_num_bk<VT, ACC, NW, U>), dim3(grid), dim3(WAVE * NW), 0, c.stream, a);
    return hipGetLastError();
}

template <typename VT, int ACC>
hipError_t num_bk_acc(const NumArgs<VT> &a, int kind, const LaunchCfg &c, int64_t rows) {
    switch (kind) {
    case K_BK0: return num_bk_u<VT, ACC, 1, 2>(a, c, rows);
    case K_BK1: return num_bk_u<VT, ACC, 1, 4>(a, c, rows);
    case K_BK2: return num_bk_u<VT, ACC, 1, 8>(a, c, rows);
    case K_BK3: return num_bk_u<VT, ACC, 2, 8>(a, c, rows);
    case K_BK4: return num_bk_u<VT, ACC, 4, 8>(a, c, rows);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_sym_bk(const SymArgs &a, int kind, const LaunchCfg &c, int64_t rows) {
    switch (kind) {
    case K_BK0: return sym_bk_u<1, 2>(a, c, rows);
    case K_BK1: return sym_bk_u<1, 4>(a, c, rows);
    case K_BK2: return sym_bk_u<1, 8>(a, c, rows);
    case K_BK3: return sym_bk_u<2, 8>(a, c, rows);
    case K_BK4: return sym_bk_u<4, 8>(a, c, rows);
    default: return hipErrorInvalidValue;
    }
}

template <>
hipError_t launch_num_bk<double>(const NumArgs<double> &a, int, int kind, const LaunchCfg &c, int64_t rows) {
    return num_bk_acc<double, ACC_NATIVE>(a, kind, c, rows);
}
template <>
hipError_t launch_num_bk<float>(const NumArgs<float> &a, int acc, int kind, const LaunchCfg &c, int64_t rows) {
    if (acc == ACC_COMP) return num_bk_acc<float, ACC_COMP>(a, kind, c, rows);
    if (acc == ACC_WIDE) return num_bk_acc<float, ACC_WIDE>(a, kind, c, rows);
    return num_bk_acc<float, ACC_NATIVE>(a, kind, c, rows);
}

}  // namespace spg
