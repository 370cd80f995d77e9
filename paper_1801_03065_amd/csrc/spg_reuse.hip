// Numeric phase on a known structure: the Reuse case of the Experiments
// section (symbolic once, numeric repeated with new values on the same
// structure), taken one step further.
//
// After a numeric call has written C's sorted columns, every multiplication
// (i, k, j) of Algorithm 1 has a fixed place in row i of C: the rank of j
// among the row's columns.  A position map -- one 16-bit rank per
// multiplication, in the row's product order (A entries in stored order, each
// B row in stored order) -- is taken once from C's columns by binary search.
// A later numeric call on new values then needs no accumulator structure at
// all (no hash, no bit window, no sort): each product is added at its rank
// in an LDS copy of the row, and only C's values are written.
//
// Work split: short rows in teams of T = 2^LGT < 64 lanes (WAVE / T rows per
// wavefront); a team stages its row's A entries T at a time (B row start and
// length, the prefix of the lengths, A's value), then groups of G = 2^LGS
// lanes walk one staged B row each.  Other rows take a wavefront, which walks
// their products flat (k_map_flat).
#include "spg_accum.hpp"
#include "spg_flat.hpp"
#include "spg_internal.hpp"

namespace spg {

namespace {

struct MapLayout {
    size_t b0, a, len, pre, vals, total;
};
__host__ __device__ inline MapLayout map_layout(int r_max, int teams, int acc_bytes) {
    MapLayout L{};
    L.b0 = 0;
    L.a = 8 * WAVE;
    L.len = 16 * WAVE;
    L.pre = 20 * WAVE;
    L.vals = 24 * WAVE;
    L.total = L.vals + align16((size_t)acc_bytes * r_max * teams);
    return L;
}

// Rows of this wavefront and team: the wavefront takes NT consecutive rows of
// its die's slice per step; the loop runs while the wavefront's first row is
// in the slice (uniform), a team whose row is past the end idles.
struct TeamRow {
    bool valid;
    int i;
    int64_t ab, ae, cb, ce, mo;
};

template <int LGT>
__device__ __forceinline__ int team_total(int inc) {
    constexpr int T = 1 << LGT;
    return __shfl(inc, T - 1, T);
}

template <int LGT, typename F>
__device__ __forceinline__ void map_rows(const RowSet &rs, const int64_t *arp, const int64_t *coff,
                                         const int64_t *moff, F &&body) {
    constexpr int T = 1 << LGT, NT = WAVE / T;
    const int l = lane_id(), team = l >> LGT;
    int64_t lo, hi;
    rs_bounds(rs, lo, hi);
    const Slice sl = xcd_slice(lo, hi, NT, 0);
    for (int64_t r0 = sl.idx; r0 < sl.end; r0 += sl.step) {
        TeamRow tr{};
        const int64_t r = r0 + team;
        tr.valid = r < sl.end;
        if (tr.valid) {
            tr.i = rs.rows[r];
            tr.ab = arp[tr.i];
            tr.ae = arp[tr.i + 1];
            tr.cb = coff[tr.i];
            tr.ce = coff[tr.i + 1];
            tr.mo = moff[tr.i];
        }
        body(tr);
    }
}

// Stage the team's A entries [e0, e0 + T) of the row: returns the team's
// total product count of the chunk; st_* hold, per lane, the entry's B row
// start, length, product offset inside the row (carry + exclusive prefix)
// and A value.
template <int LGT, typename VT>
__device__ __forceinline__ int stage_chunk(const TeamRow &tr, int64_t e0, int carry, const int32_t *aci,
                                           const VT *aval, const int64_t *brp, int64_t *st_b0, double *st_a,
                                           int *st_len, int *st_pre) {
    const int l = lane_id(), t = l & ((1 << LGT) - 1);
    const int64_t e = e0 + t;
    int64_t b0 = 0;
    int len = 0;
    double av = 0.0;
    if (tr.valid && e < tr.ae) {
        const int j = aci[e];
        b0 = brp[j];
        len = (int)(brp[j + 1] - b0);
        if (aval) av = (double)aval[e];
    }
    const int inc = team_scan<LGT>(len, t);
    st_b0[l] = b0;
    st_len[l] = len;
    st_pre[l] = carry + inc - len;
    st_a[l] = av;
    return team_total<LGT>(inc);
}

// Position map of short rows, in teams (one-time, from C's sorted columns).
template <int LGT, int LGS>
__global__ __launch_bounds__(WAVE) void k_posmap(NumArgs<double> a, const int32_t *cci) {
    constexpr int T = 1 << LGT, G = 1 << LGS, NG = T / G;
    __shared__ int64_t st_b0[WAVE];
    __shared__ double st_a[WAVE];
    __shared__ int st_len[WAVE], st_pre[WAVE];
    const int l = lane_id(), team = l >> LGT, t = l & (T - 1), g = t >> LGS, q = t & (G - 1);
    map_rows<LGT>(a.rs, a.arp, a.coff, a.map_off, [&](const TeamRow &tr) {
        const int64_t na = tr.valid ? tr.ae - tr.ab : 0;
        const int nch = wave_max((int)((na + T - 1) / T));
        int carry = 0;
        for (int c = 0; c < nch; ++c) {
            const int tot = stage_chunk<LGT, double>(tr, tr.ab + (int64_t)c * T, carry, a.aci, nullptr, a.brp,
                                                      st_b0, st_a, st_len, st_pre);
            wave_lds_sync();
            for (int s = g; s < T; s += NG) {
                const int u = team * T + s, len = st_len[u];
                const int64_t b0 = st_b0[u];
                const int64_t mb = tr.mo + st_pre[u];
                for (int p = q; p < len; p += G) {
                    const int col = a.bci[b0 + p];
                    int64_t lo2 = tr.cb, n2 = tr.ce - tr.cb;  // lower bound of col in C's row
                    while (n2 > 0) {
                        const int64_t h2 = n2 >> 1;
                        if (cci[lo2 + h2] < col) {
                            lo2 += h2 + 1;
                            n2 -= h2 + 1;
                        } else {
                            n2 = h2;
                        }
                    }
                    if (lo2 >= tr.ce || cci[lo2] != col) {
                        atomicAdd(&a.st->mismatch, 1);  // C's columns are not this product's
                        lo2 = tr.cb;
                    }
                    a.map[mb + p] = (uint16_t)(lo2 - tr.cb);
                }
            }
            carry += tot;
            wave_lds_sync();
        }
    });
}

// Rows with a wavefront each, their products walked flat, U per lane and round,
// so ranks load and store as whole cache lines and B's entries in runs, all of
// a round in flight together.  The next row's A entries and their B row
// extents, and the bounds of the row after it, load during the row.
struct FlatRow {
    int64_t ab, ae, cb, mo;
    int rn;
};

// begin(row); products(row, map of the chunk, first product, products of the
// chunk, run and B entry per product); finish(row).  Products past the chunk
// repeat its last one.  VALUES: where the B rows of a chunk have up to map_own
// entries, own(row, map of the chunk, this lane's products, their first number,
// their first B entry, A's value) takes the chunk with a lane per B row: no scan,
// staging or search.  50,000 rows of 300 A entries, B rows of one: 108 us a call
// against 191 flat, of two 154 against 203.  (With U = 1, rows of up to 64 products, a second
// entry's registers cost a wavefront per SIMD: 200,000 rows of 64 products 136 us, 93
// without.)
template <int U>
constexpr int map_own = U == 1 ? 1 : 2;
template <bool VALUES, typename VT, typename IX, int U, typename Begin, typename Own, typename Products,
          typename Finish>
__device__ __forceinline__ void flat_rows(const NumArgs<VT> &a, IX *rel, IX *off, VT *sav, uint32_t *wb, Begin &&begin,
                                          Own &&own, Products &&products, Finish &&finish) {
    const int l = lane_id();
    int64_t lo, hi;
    rs_bounds(a.rs, lo, hi);
    const Slice sl = xcd_slice(lo, hi);
    auto bounds = [&](int64_t q) {
        FlatRow r{};
        if (q < sl.end) {
            const int i = read_first(a.rs.rows[q]);
            r.ab = a.arp[i];
            r.ae = a.arp[i + 1];
            r.cb = a.coff[i];
            r.rn = (int)(a.coff[i + 1] - r.cb);
            r.mo = a.map_off[i];
        }
        return r;
    };
    int64_t p = sl.idx, b0 = 0, b1 = 0;
    FlatRow cur = bounds(p);
    VT av = VT(0);
    if (l < cur.ae - cur.ab) {
        const int j = a.aci[cur.ab + l];
        if constexpr (VALUES) av = a.aval[cur.ab + l];
        b0 = a.brp[j];
        b1 = a.brp[j + 1];
    }
    FlatRow nxt = bounds(p + sl.step);
    for (; p < sl.end; p += sl.step) {
        begin(cur);
        int nj = 0;
        VT nav = VT(0);
        const bool have = l < nxt.ae - nxt.ab;
        if (have) {
            nj = a.aci[nxt.ab + l];
            if constexpr (VALUES) nav = a.aval[nxt.ab + l];
        }
        const FlatRow after = bounds(p + 2 * sl.step);
        uint16_t *map = a.map + cur.mo;
        for (int64_t c0 = cur.ab; c0 < cur.ae; c0 += WAVE) {
            const int cn0 = (int)min((int64_t)WAVE, cur.ae - c0);
            if (c0 != cur.ab && l < cn0) {
                const int j = a.aci[c0 + l];
                if constexpr (VALUES) av = a.aval[c0 + l];
                b0 = a.brp[j];
                b1 = a.brp[j + 1];
            }
            const long long len = l < cn0 ? b1 - b0 : 0;
            if constexpr (VALUES) {
                constexpr int OWN = map_own<U>;
                if (__ballot(len > OWN) == 0) {
                    const unsigned long long first = __ballot(len > 0), second = OWN > 1 ? __ballot(len > 1) : 0;
                    own(cur, map, (int)len, mbcnt(first) + mbcnt(second), b0, av);
                    map += __popcll(first) + __popcll(second);
                    continue;
                }
            }
            const long long inc = wave_incl_scan64(len + (len > 0 ? FLAT_ONE : 0));
            const long long all = __shfl(inc, WAVE - 1);
            const IX tot = (IX)(all & FLAT_LEN);
            const int cn = (int)(all >> FLAT_SHIFT);
            wave_lds_sync();
            if (len > 0) {
                const int run = (int)(inc >> FLAT_SHIFT) - 1;
                const long long end = inc & FLAT_LEN;
                off[run] = (IX)end;
                rel[run] = (IX)(b0 - (end - len));
                if constexpr (VALUES) sav[run] = av;
            }
            wave_lds_sync();
            int kc = 0;
            for (IX F = 0; F < tot; F += (IX)(U * WAVE)) {
                int k[U], rk[U];
                IX e[U];
                if constexpr (VALUES) {  // the products' ranks, on their way during the search for their runs
#pragma unroll
                    for (int u = 0; u < U; ++u) rk[u] = map[min(F + (u * WAVE + l), tot - 1)];
                }
                kc = flat_window<U>(off, cn, F, tot, kc, wb, k);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    k[u] += kc;
                    e[u] = rel[k[u]] + min(F + (u * WAVE + l), tot - 1);
                }
                products(cur, map, F, tot, k, e, rk);
            }
            map += tot;
        }
        if (have) {
            b0 = a.brp[nj];
            b1 = a.brp[nj + 1];
        }
        wave_lds_sync();
        finish(cur);
        av = nav;
        cur = nxt;
        nxt = after;
        wave_lds_sync();
    }
}

// Values of the launch's rows on their position maps.  Bound by latency, so by
// wavefronts and loads in flight: r_max (the longest row of the launch) sizes
// the LDS.  Batch of 48 random products, FP32 (6.1e8 products): 2.5 ms, its
// data unit 75 to 91% busy; with lane groups per B row and one load in flight
// 3.7 ms.
template <typename VT, int ACC, typename IX, int U>
__global__ __launch_bounds__(WAVE) void k_map_flat(NumArgs<VT> a) {
    using Acc = Accum<VT, ACC>;
    using S = typename Acc::store_t;
    extern __shared__ __align__(16) unsigned char smem[];
    S *vals = (S *)smem;
    __shared__ IX rel[WAVE], off[WAVE];  // per staged run (see spg_flat.hpp)
    __shared__ VT sav[WAVE];
    __shared__ __align__(8) uint32_t wb[2 * U];
    const int l = lane_id();
    for (int u = l; u < a.r_max; u += WAVE) vals[u] = Acc::zero();
    const int64_t cbase = a.cbase_row >= 0 ? a.coff[a.cbase_row] : 0;
    auto rlast = [&](const FlatRow &r) { return max(min(r.rn, a.r_max) - 1, 0); };
    flat_rows<true, VT, IX, U>(
        a, rel, off, sav, wb, [](const FlatRow &) {},
        [&](const FlatRow &r, const uint16_t *map, int len, int at, int64_t e, VT av) {
            constexpr int OWN = map_own<U>;
            int rk[OWN] = {};
            VT bv[OWN] = {};
#pragma unroll
            for (int q = 0; q < OWN; ++q)
                if (q < len) {
                    rk[q] = map[at + q];
                    bv[q] = a.bval[e + q];
                }
#pragma unroll
            for (int q = 0; q < OWN; ++q)
                if (q < len) Acc::add(&vals[min(rk[q], rlast(r))], av, bv[q]);
        },
        [&](const FlatRow &r, const uint16_t *, IX F, IX tot, int (&k)[U], IX (&e)[U], int (&rk)[U]) {
            VT bv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) bv[u] = a.bval[e[u]];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (F + (u * WAVE + l) < tot) Acc::add(&vals[min(rk[u], rlast(r))], sav[k[u]], bv[u]);
        },
        [&](const FlatRow &r) {
            for (int u = l; u < min(r.rn, a.r_max); u += WAVE) {
                store_c(&a.cval[r.cb - cbase + u], Acc::fin(vals[u]));
                vals[u] = Acc::zero();
            }
        });
}

// Position map of the launch's rows (one-time, from C's sorted columns cci): a
// row's columns staged in LDS, padded to a power of two, and the searches of a
// round advanced together.  r_max: entries the dynamic LDS holds (longer rows
// cannot occur: the launch's longest row sizes it).  Batch of 48 random
// products: 4.4 ms; a search per lane in HBM took 13.4 ms.
template <typename IX, int U>
__global__ __launch_bounds__(WAVE) void k_posmap_flat(NumArgs<double> a, const int32_t *cci) {
    extern __shared__ __align__(16) unsigned char smem[];
    int32_t *cols = (int32_t *)smem;
    __shared__ IX rel[WAVE], off[WAVE];
    __shared__ __align__(8) uint32_t wb[2 * U];
    const int l = lane_id();
    int half = 0;  // the search runs over 2 * half - 1 entries
    flat_rows<false, double, IX, U>(
        a, rel, off, (double *)nullptr, wb,
        [&](const FlatRow &r) {
            half = 1;
            while (2 * half <= r.rn && 4 * half <= a.r_max) half *= 2;
            for (int t = l; t < 2 * half; t += WAVE) cols[t] = t < r.rn ? cci[r.cb + t] : INT_MAX;
        },
        [](const FlatRow &, uint16_t *, int, int, int64_t, double) {},
        [&](const FlatRow &, uint16_t *map, IX F, IX tot, int (&)[U], IX (&e)[U], int (&)[U]) {
            int c[U], at[U];
#pragma unroll
            for (int u = 0; u < U; ++u) c[u] = a.bci[e[u]];
#pragma unroll
            for (int u = 0; u < U; ++u) at[u] = 0;
            for (int s = half; s > 0; s >>= 1)
#pragma unroll
                for (int u = 0; u < U; ++u) at[u] += cols[at[u] + s - 1] < c[u] ? s : 0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (F + (u * WAVE + l) >= tot) continue;
                if (cols[at[u]] != c[u]) {
                    atomicAdd(&a.st->mismatch, 1);  // C's columns are not this product's
                    at[u] = 0;
                }
                map[F + (u * WAVE + l)] = (uint16_t)at[u];
            }
        },
        [](const FlatRow &) {});
}

// The same for short rows, in teams.  Their values are stored through the L2,
// whose lines several rows share (8 entries a row: 235 us, 247 streamed).
template <typename VT, int ACC, int LGT, int LGS>
__global__ __launch_bounds__(WAVE) void k_num_map(NumArgs<VT> a) {
    using Acc = Accum<VT, ACC>;
    using S = typename Acc::store_t;
    constexpr int T = 1 << LGT, NT = WAVE / T, G = 1 << LGS, NG = T / G;
    extern __shared__ __align__(16) unsigned char smem[];
    const MapLayout L = map_layout(a.r_max, NT, sizeof(S));
    int64_t *st_b0 = (int64_t *)(smem + L.b0);
    double *st_a = (double *)(smem + L.a);
    int *st_len = (int *)(smem + L.len), *st_pre = (int *)(smem + L.pre);
    const int l = lane_id(), team = l >> LGT, t = l & (T - 1), g = t >> LGS, q = t & (G - 1);
    S *tv = (S *)(smem + L.vals) + (size_t)team * a.r_max;
    for (int u = t; u < a.r_max; u += T) tv[u] = Acc::zero();
    const int64_t cbase = a.cbase_row >= 0 ? a.coff[a.cbase_row] : 0;
    wave_lds_sync();
    map_rows<LGT>(a.rs, a.arp, a.coff, a.map_off, [&](const TeamRow &tr) {
        const int64_t na = tr.valid ? tr.ae - tr.ab : 0;
        const int rs = tr.valid ? (int)(tr.ce - tr.cb) : 0;
        const int rlast = rs > 0 ? rs - 1 : 0;
        const int nch = wave_max((int)((na + T - 1) / T));
        int carry = 0;
        for (int c = 0; c < nch; ++c) {
            const int tot = stage_chunk<LGT, VT>(tr, tr.ab + (int64_t)c * T, carry, a.aci, a.aval, a.brp, st_b0,
                                                  st_a, st_len, st_pre);
            wave_lds_sync();
            if (rs > 0) {
                for (int s = g; s < T; s += NG) {
                    const int u = team * T + s, len = st_len[u];
                    const int64_t b0 = st_b0[u];
                    const int64_t mb = tr.mo + st_pre[u];
                    const VT av = (VT)st_a[u];
                    for (int p = q; p < len; p += G) {
                        const int rk = min((int)a.map[mb + p], rlast);
                        Acc::add(&tv[rk], av, a.bval[b0 + p]);
                    }
                }
            }
            carry += tot;
            wave_lds_sync();
        }
        for (int u = t; u < rs; u += T) {
            a.cval[tr.cb - cbase + u] = Acc::fin(tv[u]);
            tv[u] = Acc::zero();
        }
        wave_lds_sync();
    });
}

template <int LGT, int LGS>
hipError_t posmap_ts(const NumArgs<double> &a, const int32_t *cci, const LaunchCfg &c, int64_t rows) {
    constexpr int NT = WAVE >> LGT;
    int grid = resident_grid(k_posmap<LGT, LGS>, WAVE, 0, c.cus);
    const int64_t need = (rows + NT - 1) / NT;
    grid = (int)std::min<int64_t>(grid, std::max<int64_t>(XCDS, ((need + XCDS - 1) / XCDS) * XCDS));
    hipLaunchKernelGGL((k_posmap<LGT, LGS>), dim3(grid), dim3(WAVE), 0, c.stream, a, cci);
    return hipGetLastError();
}

template <typename VT, int ACC, int LGT, int LGS>
hipError_t num_map_ts(const NumArgs<VT> &a, const LaunchCfg &c, int64_t rows) {
    using S = typename Accum<VT, ACC>::store_t;
    constexpr int NT = WAVE >> LGT;
    const size_t lds = map_layout(a.r_max, NT, sizeof(S)).total;
    int grid = resident_grid(k_num_map<VT, ACC, LGT, LGS>, WAVE, lds, c.cus);
    const int64_t need = (rows + NT - 1) / NT;
    grid = (int)std::min<int64_t>(grid, std::max<int64_t>(XCDS, ((need + XCDS - 1) / XCDS) * XCDS));
    hipLaunchKernelGGL((k_num_map<VT, ACC, LGT, LGS>), dim3(grid), dim3(WAVE), lds, c.stream, a);
    return hipGetLastError();
}

// lanes per B row: 1 .. T
template <int LGT, typename F>
hipError_t by_lgs(int lgs, F &&f) {
    lgs = std::max(0, std::min(lgs, LGT));
    switch (lgs) {
    case 0: return f(std::integral_constant<int, 0>{});
    case 1: return f(std::integral_constant<int, 1>{});
    case 2: return f(std::integral_constant<int, 2>{});
    case 3: return f(std::integral_constant<int, (LGT >= 3 ? 3 : 2)>{});
    case 4: return f(std::integral_constant<int, (LGT >= 4 ? 4 : 2)>{});
    case 5: return f(std::integral_constant<int, (LGT >= 5 ? 5 : 2)>{});
    default: return f(std::integral_constant<int, 2>{});
    }
}

template <typename F>
hipError_t by_team(int lgt, F &&f) {  // teams of less than a wavefront
    switch (lgt) {
    case 4: return f(std::integral_constant<int, 4>{});
    case 5: return f(std::integral_constant<int, 5>{});
    default: return f(std::integral_constant<int, 3>{});
    }
}

template <typename IX>
hipError_t posmap_flat(NumArgs<double> a, const int32_t *cci, const LaunchCfg &c, int64_t rows) {
    int r = 2 * WAVE;
    while (r <= a.r_max) r *= 2;
    a.r_max = r;
    int grid = resident_grid(k_posmap_flat<IX, 4>, WAVE, 4 * (size_t)r, c.cus);
    grid = (int)std::min<int64_t>(grid, std::max<int64_t>(XCDS, ((rows + XCDS - 1) / XCDS) * XCDS));
    hipLaunchKernelGGL((k_posmap_flat<IX, 4>), dim3(grid), dim3(WAVE), 4 * (size_t)r, c.stream, a, cci);
    return hipGetLastError();
}

template <typename VT, int ACC, typename IX, int U>
hipError_t map_flat_u(const NumArgs<VT> &a, const LaunchCfg &c, int64_t rows) {
    const size_t lds = align16(sizeof(typename Accum<VT, ACC>::store_t) * (size_t)a.r_max);
    int grid = resident_grid(k_map_flat<VT, ACC, IX, U>, WAVE, lds, c.cus);
    grid = (int)std::min<int64_t>(grid, std::max<int64_t>(XCDS, ((rows + XCDS - 1) / XCDS) * XCDS));
    hipLaunchKernelGGL((k_map_flat<VT, ACC, IX, U>), dim3(grid), dim3(WAVE), lds, c.stream, a);
    return hipGetLastError();
}

// Products per lane and round by the largest kind of the launch: most rows then
// take one or two rounds (20000 rows of 100 to 150 products, FP64: 49.5 us a
// call with 4, 52 with 2 or 8; 125,000 rows of 62: 52 us with 1, 59 with 2, 53 in
// teams of 64 lanes).  32-bit product numbers where 64 A entries cannot form
// 2^31 products.
template <typename VT, int ACC>
hipError_t map_flat(const NumArgs<VT> &a, const LaunchCfg &c, int64_t rows) {
    const int last = a.rs.kind + a.rs.more;
    const bool i32 = flat_32bit(a.nnzb, WAVE, 8 * WAVE);
    if (last == K_SR)
        return i32 ? map_flat_u<VT, ACC, int32_t, 1>(a, c, rows) : map_flat_u<VT, ACC, int64_t, 1>(a, c, rows);
    if (last == K_BK0)
        return i32 ? map_flat_u<VT, ACC, int32_t, 2>(a, c, rows) : map_flat_u<VT, ACC, int64_t, 2>(a, c, rows);
    if (last == K_BK1 || last == K_BK2)
        return i32 ? map_flat_u<VT, ACC, int32_t, 4>(a, c, rows) : map_flat_u<VT, ACC, int64_t, 4>(a, c, rows);
    return i32 ? map_flat_u<VT, ACC, int32_t, 8>(a, c, rows) : map_flat_u<VT, ACC, int64_t, 8>(a, c, rows);
}

template <typename VT, int ACC>
hipError_t num_map_acc(const NumArgs<VT> &a, int lgt, int lgs, const LaunchCfg &c, int64_t rows) {
    if (lgt >= 6) return map_flat<VT, ACC>(a, c, rows);
    return by_team(lgt, [&](auto T) {
        constexpr int LT = decltype(T)::value;
        return by_lgs<LT>(lgs, [&](auto S) {
            constexpr int LS = decltype(S)::value;
            return num_map_ts<VT, ACC, LT, LS>(a, c, rows);
        });
    });
}

}  // namespace


hipError_t launch_posmap(const NumArgs<double> &a, const int32_t *cci, int lgt, int lgs, const LaunchCfg &c,
                         int64_t rows) {
    if (lgt >= 6)
        return flat_32bit(a.nnzb, WAVE, 4 * WAVE) ? posmap_flat<int32_t>(a, cci, c, rows)
                                                  : posmap_flat<int64_t>(a, cci, c, rows);
    return by_team(lgt, [&](auto T) {
        constexpr int LT = decltype(T)::value;
        return by_lgs<LT>(lgs, [&](auto S) {
            constexpr int LS = decltype(S)::value;
            return posmap_ts<LT, LS>(a, cci, c, rows);
        });
    });
}

template <>
hipError_t launch_num_map<double>(const NumArgs<double> &a, int, int lgt, int lgs, const LaunchCfg &c, int64_t rows) {
    return num_map_acc<double, ACC_NATIVE>(a, lgt, lgs, c, rows);
}
template <>
hipError_t launch_num_map<float>(const NumArgs<float> &a, int acc, int lgt, int lgs, const LaunchCfg &c, int64_t rows) {
    if (acc == ACC_COMP) return num_map_acc<float, ACC_COMP>(a, lgt, lgs, c, rows);
    if (acc == ACC_WIDE) return num_map_acc<float, ACC_WIDE>(a, lgt, lgs, c, rows);
    return num_map_acc<float, ACC_NATIVE>(a, lgt, lgs, c, rows);
}

}  // namespace spg

namespace spg {

namespace {

// Multiplications per row of the rows that get a position map (rows of the
// wavefront and team kinds in the plan's main or FP64-accumulated lists),
// 0 for the others.
__global__ __launch_bounds__(256) void k_map_rows(int64_t m, const uint8_t *kind, const uint8_t *kind_heavy,
                                                  const int64_t *rflops, int32_t *out) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < m; i += (int64_t)gridDim.x * 256) {
        const int k = kind[i], kh = kind_heavy ? kind_heavy[i] : 0;
        const bool mapped = map_kind(k) || map_kind(kh);
        out[i] = mapped ? (int32_t)rflops[i] : 0;
    }
}

}  // namespace

hipError_t launch_map_rows(int64_t m, const uint8_t *kind, const uint8_t *kind_heavy, const int64_t *rflops,
                           int32_t *out, hipStream_t s) {
    if (m == 0) return hipSuccess;
    const int g = (int)std::min<int64_t>(4096, (m + 255) / 256);
    hipLaunchKernelGGL(k_map_rows, dim3(g), dim3(256), 0, s, m, kind, kind_heavy, rflops, out);
    return hipGetLastError();
}

}  // namespace spg
