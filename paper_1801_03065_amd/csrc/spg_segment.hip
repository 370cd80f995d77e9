// Heavy rows in column segments: the dense accumulator of the Accumulators
// subsection, cut to the size of LDS.
//
// A heavy row of C (thousands to a million entries spread over up to 2^20
// columns) does not fit in LDS as a whole.  The symbolic phase, which holds
// the row's complete bit window, cuts it into segments: runs of consecutive
// column-set words with at most SG_CAP entries that stay inside one aligned
// group of SG_NW words.  The numeric phase then walks the segments in column
// order, one 512-lane workgroup per row (a launch may hold two row sets, the
// second taken first and accumulated with its own accumulator):
//
//   1. the part of each B row that falls in the segment (B's columns are
//      sorted, so it is one run; each A entry keeps a cursor into its B row
//      from segment to segment, in a register for rows of one chunk of A
//      entries, in HBM scratch for longer rows, else binary search); the
//      nonempty runs are staged back to back,
//   2. structure: the segment's words, as the symbolic phase kept them, else
//      the runs' columns OR-ed into an LDS bit array over the words,
//      Thread-Flat-Parallel over the segment's products (spg_flat.hpp); the
//      bits must be as many as the plan's entries,
//   3. ranks: prefix popcounts of the words give every column its place in
//      the row,
//   4. values: each product added at its rank in LDS (Algorithm 1's
//      accumulation), Thread-Flat-Parallel again,
//   5. write-out: values in rank order, then columns expanded from the bits
//      into LDS and stored in rank order (both coalesced), at the segment's
//      offset in the row, which the symbolic phase recorded.
//
// Kept words may not be the products' (B changed behind the plan).  They are if
// every product finds its bit and every entry has a product; an entry without
// one still holds the -0.0 it starts from, which sums that cancel do not give.
// So a row whose products all found their bits and that has no entry of -0.0 is
// done (one more instruction per product, two per entry: R-MAT scale 17 and 15
// unchanged within 1%); an entry of -0.0 (products of -0.0 only: stored zeros)
// has the row's bits OR-ed and counted after all, a product without its bit has
// the row done again on the words of its products.
//
// Nothing lives in HBM but the inputs, the kept words and C; a row with one
// segment (its entries and window fit) runs the same steps once, with whole B
// rows.
//
// Bound by the vector-memory path (its data unit 65% busy before the words were
// kept: runs inside a segment are a few entries, so a 64-lane load touches 16
// cache lines) and by latency at 16 wavefronts per CU.  Keeping the words saves
// the OR walk, half the loads and half the owner searches.  R-MAT scale 17
// squared, FP64 (3.5e9 multiplications): 20.8 -> 14.0 ms, 4.0 ps a
// multiplication; scale 20, where the words (over 40 GB) are rebuilt: 611 ->
// 526 ms, symbolic phase 166 -> 121 ms.
#include "spg_accum.hpp"
#include "spg_flat.hpp"
#include "spg_internal.hpp"

namespace spg {
namespace {

constexpr int SG_U = 8;  // products per lane per round of the flat walks (loads in flight)
// Lanes per workgroup (one heavy row).  LDS (47 to 67 KB) and registers allow two
// workgroups per CU; 512 lanes rather than 256 double the loads in flight per CU for the
// same LDS, with registers held to 128 (4 waves per SIMD).
constexpr int SG_WG = 512;

__device__ __forceinline__ long long sg_block_excl_scan(long long v, long long *red, long long *total) {
    const int t = threadIdx.x, l = lane_id(), wv = t / WAVE;
    const long long inc = wave_incl_scan64(v);
    __syncthreads();
    if (l == WAVE - 1) red[wv] = inc;
    __syncthreads();
    long long off = 0, tot = 0;
#pragma unroll
    for (int u = 0; u < SG_WG / WAVE; ++u) {
        const long long x = red[u];
        if (u < wv) off += x;
        tot += x;
    }
    *total = tot;
    return off + inc - v;
}

__device__ __forceinline__ int sg_next_row(const RowSet &rs, int64_t lo, int64_t hi, int &x, long long *red) {
    __syncthreads();
    if (threadIdx.x == 0) {
        const int64_t t = xcd_grab(rs.queue, lo, hi, x);
        red[SG_WG / WAVE] = t < 0 ? -1 : rs.rows[t];
        red[SG_WG / WAVE + 1] = x;
    }
    __syncthreads();
    x = read_first((int)red[SG_WG / WAVE + 1]);
    return read_first((int)red[SG_WG / WAVE]);  // scalar: the row's bounds then live in scalar registers
}

// First index in [lo, hi) whose column is >= key (hi when none); the row's
// columns are sorted.  The two ends are tested first: runs that start at the
// row's start or end at its end need no search.
__device__ __forceinline__ int64_t sg_lower_bound(const int32_t *bci, int64_t lo, int64_t hi, int64_t key) {
    if (lo >= hi || (int64_t)bci[lo] >= key) return lo;
    if ((int64_t)bci[hi - 1] < key) return hi;
    ++lo;  // bci[lo] < key
    --hi;  // bci[hi] >= key
    while (lo < hi) {
        const int64_t mid = lo + ((hi - lo) >> 1);
        if ((int64_t)bci[mid] < key) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// First index in [lo, hi) whose column is >= key, searched from lo (the run
// is usually short): four entries in one load, which the products then find in
// the cache; beyond them jumps of 4, 8, 16, ... and a binary search in the last
// one.  (Testing the row's last entry first cost a line of its own per A entry
// and segment: R-MAT scale 17 18.46 -> 18.22 ms, scale 15, FP32 numeric, 1.73 ->
// 1.69.)
__device__ __forceinline__ int64_t sg_gallop(const int32_t *bci, int64_t lo, int64_t hi, int64_t key) {
    if (hi - lo > 4) {
        struct Four {
            int32_t a, b, c, d;
        };
        const Four q = *(const Four *)&bci[lo];
        const int r = (q.a < key) + (q.b < key) + (q.c < key) + (q.d < key);
        if (r < 4) return lo + r;
        lo += 4;
        int64_t step = 4;
        for (; lo + step < hi; step <<= 1) {
            if ((int64_t)bci[lo + step - 1] >= key) {
                hi = lo + step - 1;
                break;
            }
            lo += step;
        }
        while (hi - lo > 4) {
            const int64_t mid = lo + ((hi - lo) >> 1);
            if ((int64_t)bci[mid] < key) lo = mid + 1;
            else hi = mid;
        }
    }
    int r = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (lo + k < hi) r += (int64_t)bci[lo + k] < key;
    return lo + r;
}

// An accumulator without a product: -0.0, which adding any product replaces
// (with that product; +0.0 by a sum of zero).
__device__ __forceinline__ double sg_none(double) { return -0.0; }
__device__ __forceinline__ float sg_none(float) { return -0.0f; }
__device__ __forceinline__ unsigned long long sg_none(unsigned long long) { return 0x80000000ull; }  // (s, c)
__device__ __forceinline__ bool sg_is_none(double v) { return __double_as_longlong(v) == LLONG_MIN; }
__device__ __forceinline__ bool sg_is_none(float v) { return __float_as_int(v) == INT_MIN; }
__device__ __forceinline__ bool sg_is_none(unsigned long long v) { return (int)(uint32_t)v == INT_MIN; }

// ACC accumulates the rows of a.rs, ACC2 those of a.rs2 (FP32 values: the
// heaviest rows in FP64); the value array holds either kind of entry.  IX:
// 32-bit B indices where byte offsets into B's values fit 32 bits.
template <typename VT, int ACC, int ACC2, typename IX>
__global__ __launch_bounds__(SG_WG) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_num_sg(NumArgs<VT> a) {
    using A = Accum<VT, ACC>;
    using S = typename A::store_t;
    using A2 = Accum<VT, ACC2>;
    using S2 = typename A2::store_t;
    constexpr int VB = sizeof(S) > sizeof(S2) ? sizeof(S) : sizeof(S2);
    __shared__ __align__(16) uint32_t bits[SG_NW];
    __shared__ uint16_t pre[SG_NW];
    __shared__ __align__(16) unsigned char vals_raw[SG_CAP * VB];
    S *vals = (S *)vals_raw;
    S2 *vals2 = (S2 *)vals_raw;
    __shared__ IX st_rel[SG_WG];   // per nonempty run: its first B entry, less its first product
    __shared__ int st_off[SG_WG];  // inclusive prefix of the run lengths
    __shared__ VT st_a[SG_WG];
    __shared__ long long red[SG_WG / WAVE + 2];
    __shared__ __align__(8) uint32_t wb[SG_WG / WAVE][2 * SG_U];  // flat_window's scratch per wavefront
    __shared__ int redo_none, redo_miss;  // kept words: an entry may have no product, a product's column is not in them
    const int t = threadIdx.x, l = lane_id(), wv = read_first(t / WAVE);
    for (int w = t; w < SG_NW; w += SG_WG) bits[w] = 0;
    int64_t qlo, qhi;
    rs_bounds(a.rs, qlo, qhi);
    const int64_t cbase = a.cbase_row >= 0 ? a.coff[a.cbase_row] : 0;
    int x = blockIdx.x % XCDS;
    // a second row set (the heaviest rows) is drained first, then the first set
    bool second = a.rs2.rows != nullptr;
    int64_t qlo2 = 0, qhi2 = 0;
    if (second) rs_bounds(a.rs2, qlo2, qhi2);
    int x2 = x;
    enum { NO, PRODUCTS, CHECK };  // the row again, on the words of its products (CHECK: to count them)
    int again = NO, i = 0;
    // the first n accumulators of the current row set
    auto clear = [&](int n) {
        if (ACC2 != ACC && second)
            for (int r = t; r < n; r += SG_WG) vals2[r] = sg_none(S2());
        else
            for (int r = t; r < n; r += SG_WG) vals[r] = sg_none(S());
    };
    clear(SG_CAP);
    for (;;) {
        if (again != NO) {  // values may have been added past the segment's
            clear(SG_CAP);
            __syncthreads();
        } else if (second) {
            i = sg_next_row(a.rs2, qlo2, qhi2, x2, red);
            if (i < 0) {
                second = false;
                clear(SG_CAP);
                continue;
            }
        } else {
            i = sg_next_row(a.rs, qlo, qhi, x, red);
            if (i < 0) break;
        }
        if (t == 0) redo_none = redo_miss = 0;
        const bool acc2 = ACC2 != ACC && second;  // this row accumulates with ACC2
        const int2 win = a.rwin[i];
        const int wlo = win.x, nw = win.y - win.x + 1;
        const int64_t c0 = a.coff[i], nnz = a.coff[i + 1] - c0;
        const int64_t ab = a.arp[i], ae = a.arp[i + 1];
        const bool has_list = a.plan_len != nullptr && a.sym_kind[i] == K_DG && a.plan_len[i] > 0;
        const uint2 *list = has_list ? a.plan + a.plan_off[i] : nullptr;
        const uint32_t *kept = again == NO && has_list && a.sgb != nullptr && a.sgb_len[i] > 0 ? a.sgb + a.sgb_off[i] : nullptr;
        const int nseg = has_list ? read_first((int)list[0].x) : 1;
        const bool single = nseg == 1;
        const bool one_chunk = ae - ab <= SG_WG;
        // several chunks: per A entry, in this workgroup's scratch, the B
        // entry where its run in the segment starts (cursor), where that run
        // ends, and the end of its B row (absolute positions: nnz(B) < 2^31),
        // so that a chunk's staging loads no A column and no B row extent
        int32_t *cur_g = nullptr, *nxt_g = nullptr, *end_g = nullptr;
        if (!one_chunk && !single && a.sg_cur != nullptr && ae - ab <= a.sg_cap) {
            cur_g = a.sg_cur + (int64_t)blockIdx.x * 3 * a.sg_cap;
            nxt_g = cur_g + a.sg_cap;
            end_g = nxt_g + a.sg_cap;
            for (int64_t k = t; k < ae - ab; k += SG_WG) {
                const int j = a.aci[ab + k];
                cur_g[k] = (int32_t)a.brp[j];
                end_g[k] = (int32_t)a.brp[j + 1];
            }
            __syncthreads();
        }
        // one chunk: lane t keeps A entry t for the whole row, with a cursor
        // into its B row that moves from segment to segment
        int64_t cur = 0, bend = 0;
        VT av1 = VT(0);
        if (one_chunk && ab + t < ae) {
            const int j = a.aci[ab + t];
            cur = a.brp[j];
            bend = a.brp[j + 1];
            av1 = a.aval[ab + t];
        }
        int bad = 0;
        for (int sg = 0; sg < nseg; ++sg) {
            int w1 = 0, w2 = nw;
            int64_t p1 = 0, p2 = nnz;
            if (has_list) {
                const uint2 d1 = list[1 + sg], d2 = list[2 + sg];
                w1 = read_first((int)d1.x);
                p1 = (uint32_t)read_first((int)d1.y);
                w2 = read_first((int)d2.x);
                p2 = (uint32_t)read_first((int)d2.y);
            }
            const int cnt = (int)(p2 - p1);
            const int64_t col_lo = (int64_t)(wlo + w1) << 5, col_hi = (int64_t)(wlo + w2) << 5;
            const int span = min(w2 - w1, SG_NW);
            const int dbase = wlo + w1;  // column-set word of bits[0]
            // Stage the nonempty runs of one chunk of A entries, back to back:
            // returns their number, *tot products.  A run lies in the segment's
            // words, which bounds it (and a chunk's products below 2^31).
            // first / last: the first and last walk over the segment's runs.
            auto stage = [&](int64_t cb, bool first, bool last, int *tot) -> int {
                int64_t s0 = 0, s1 = 0;
                VT av = VT(0);
                if (one_chunk) {
                    s0 = cur;
                    if (ab + t < ae) s1 = sg + 1 == nseg ? bend : sg_gallop(a.bci, cur, bend, col_hi);
                    else s1 = s0;
                    cur = s1;
                    av = av1;
                } else if (cb + t < ae) {
                    const int64_t k = cb - ab + t;
                    if (cur_g) {
                        s0 = cur_g[k];
                        if (first) {
                            s1 = end_g[k];
                            if (sg + 1 < nseg) s1 = sg_gallop(a.bci, s0, s1, col_hi);
                            if (!last) nxt_g[k] = (int32_t)s1;
                        } else {
                            s1 = nxt_g[k];
                        }
                        if (last) cur_g[k] = (int32_t)s1;  // the next segment starts where this run ends
                    } else {
                        const int j = a.aci[cb + t];
                        s0 = a.brp[j];
                        s1 = a.brp[j + 1];
                        if (!single) {
                            s0 = sg_lower_bound(a.bci, s0, s1, col_lo);
                            s1 = sg_lower_bound(a.bci, s0, s1, col_hi);
                        }
                    }
                    av = a.aval[cb + t];
                }
                const long long len = min(s1 - s0, (int64_t)SG_NW * 32);
                long long all;
                const long long ex = sg_block_excl_scan(len + (len > 0 ? FLAT_ONE : 0), red, &all);
                if (len > 0) {
                    const int k = (int)(ex >> FLAT_SHIFT), before = (int)(ex & FLAT_LEN);
                    st_rel[k] = (IX)(s0 - before);
                    st_off[k] = before + (int)len;
                    st_a[k] = av;
                }
                *tot = read_first((int)(all & FLAT_LEN));
                __syncthreads();
                return read_first((int)(all >> FLAT_SHIFT));
            };
            // The staged products, SG_U per lane and round: body(u, product's
            // run, B entry, in range) is called in two steps, loads then use.
            auto walk = [&](int cn, int tot, auto &&use) {
                int kc = 0;
                for (int F = wv * (SG_U * WAVE); F < tot; F += SG_U * SG_WG) {
                    int k[SG_U];
                    IX e[SG_U];
                    kc = flat_window<SG_U>(st_off, cn, F, tot, kc, wb[wv], k);
#pragma unroll
                    for (int u = 0; u < SG_U; ++u) {
                        const int f = F + u * WAVE + l;
                        k[u] += kc;
                        e[u] = f < tot ? st_rel[k[u]] + f : IX(-1);
                    }
                    use(k, e);
                }
            };
            auto ldc = [&](IX e) -> int { return sizeof(IX) == 4 ? ld32(a.bci, (uint32_t)e) : a.bci[e]; };
            auto ldv = [&](IX e) -> VT { return sizeof(IX) == 4 ? ld32(a.bval, (uint32_t)e) : a.bval[e]; };
            int tot1 = 0, cn1 = 0;
            if (kept) {  // structure: as the symbolic phase stored it
                for (int w = t; w < span; w += SG_WG) bits[w] = kept[w1 + w];
                if (one_chunk) cn1 = stage(ab, true, true, &tot1);
                else __syncthreads();
            } else {
                if (one_chunk) cn1 = stage(ab, true, true, &tot1);
                for (int64_t cb = ab; cb < ae; cb += SG_WG) {
                    int tot = tot1, cn = cn1;
                    if (!one_chunk) cn = stage(cb, true, false, &tot);
                    walk(cn, tot, [&](int (&)[SG_U], IX (&e)[SG_U]) {
                        int c[SG_U];
#pragma unroll
                        for (int u = 0; u < SG_U; ++u) c[u] = ldc(max(e[u], IX(0)));
#pragma unroll
                        for (int u = 0; u < SG_U; ++u) {
                            const int d = (c[u] >> 5) - dbase;
                            if (e[u] >= 0 && (unsigned)d < (unsigned)SG_NW) atomicOr(&bits[d], 1u << (c[u] & 31));
                        }
                    });
                    if (!one_chunk) __syncthreads();  // st_* are refilled for the next chunk
                }
                __syncthreads();
            }
            {  // ranks: lane t scans words [t * SG_NW / SG_WG, ...) of the segment
                constexpr int WPL = SG_NW / SG_WG;
                const int wb = t * WPL;
                uint32_t w[WPL];
                int sum = 0;
#pragma unroll
                for (int u = 0; u < WPL; u += 4) {
                    const uint4 q = *(const uint4 *)&bits[wb + u];
                    w[u] = q.x;
                    w[u + 1] = q.y;
                    w[u + 2] = q.z;
                    w[u + 3] = q.w;
                }
#pragma unroll
                for (int u = 0; u < WPL; ++u) sum += __popc(w[u]);
                long long tot;
                int run = (int)sg_block_excl_scan(sum, red, &tot);
#pragma unroll
                for (int u = 0; u < WPL; ++u) {
                    pre[wb + u] = (uint16_t)min(run, 65535);
                    run += __popc(w[u]);
                }
                if (tot != cnt) bad = 1;
                __syncthreads();
            }
            if (again == CHECK) {  // the values stand
                if (!one_chunk) {  // past the segment (below: the walk over the values does it)
                    int tot;
                    for (int64_t cb = ab; cb < ae; cb += SG_WG) stage(cb, false, true, &tot);
                }
                for (int w = t; w < SG_NW; w += SG_WG) bits[w] = 0;
                __syncthreads();
                continue;
            }
            // values: each product added at its rank
            uint32_t hit = 1;  // bit 0: every product's column is in the words
            for (int64_t cb = ab; cb < ae; cb += SG_WG) {
                int tot = tot1, cn = cn1;
                if (!one_chunk) cn = stage(cb, kept != nullptr, true, &tot);
                walk(cn, tot, [&](int (&k)[SG_U], IX (&e)[SG_U]) {
                    int c[SG_U], r[SG_U];  // columns, ranks
                    VT v[SG_U];
#pragma unroll
                    for (int u = 0; u < SG_U; ++u) c[u] = ldc(max(e[u], IX(0)));
#pragma unroll
                    for (int u = 0; u < SG_U; ++u) v[u] = ldv(max(e[u], IX(0)));
#pragma unroll
                    for (int u = 0; u < SG_U; ++u) {
                        const int d = (c[u] >> 5) - dbase;
                        const bool in = e[u] >= 0 && (unsigned)d < (unsigned)SG_NW;
                        const uint32_t w = in ? bits[d] : ~0u;
                        const int b = c[u] & 31;
                        r[u] = in ? (int)pre[d] + bits_below(w, b) : SG_CAP;
                        hit &= w >> b;
                    }
                    if (acc2) {
#pragma unroll
                        for (int u = 0; u < SG_U; ++u)
                            if (r[u] < SG_CAP) A2::add(&vals2[r[u]], st_a[k[u]], v[u]);
                    } else {
#pragma unroll
                        for (int u = 0; u < SG_U; ++u)
                            if (r[u] < SG_CAP) A::add(&vals[r[u]], st_a[k[u]], v[u]);
                    }
                });
                if (!one_chunk) __syncthreads();  // st_* are refilled for the next chunk
            }
            __syncthreads();
            // write-out at the segment's offset, both arrays in rank order with
            // coalesced stores: first the values; then the columns, expanded
            // from the bits (one word per lane) into the freed value array;
            // the bits and values are cleared for the next segment
            const int64_t o = c0 + p1 - cbase;
            const int cw = min(cnt, SG_CAP);
            bool none = false;
            auto put = [&](const auto *from, auto fin) {
                for (int r = t; r < cw; r += SG_WG) {
                    none |= sg_is_none(from[r]);
                    store_c(&a.cval[o + r], fin(from[r]) + VT(0));  // (-0.0 becomes 0.0)
                }
            };
            if (acc2) put(vals2, A2::fin);
            else put(vals, A::fin);
            if (none) redo_none = 1;
            if (!(hit & 1u)) redo_miss = 1;
            __syncthreads();
            int32_t *colbuf = (int32_t *)vals_raw;  // SG_CAP * VB >= 4 * SG_CAP bytes
            // (other products than the plan's reach past the segment's words and entries)
            const int wend = bad ? SG_NW : span, rend = bad ? SG_CAP : cw;
            for (int w = t; w < wend; w += SG_WG) {
                uint32_t m = bits[w];
                int r = pre[w];
                const int colb = (dbase + w) << 5;
                while (m) {
                    const int b = __ffs(m) - 1;
                    m &= m - 1;
                    if (r < cw) colbuf[r] = colb + b;
                    ++r;
                }
                bits[w] = 0;
            }
            __syncthreads();
            for (int r = t; r < cw; r += SG_WG) store_c(&a.cci[o + r], colbuf[r]);
            __syncthreads();
            clear(rend);
            __syncthreads();
        }
        if (kept) {
            const int miss = read_first(redo_miss);
            if (miss | read_first(redo_none)) again = miss ? PRODUCTS : CHECK;
        } else {
            again = NO;
        }
        if (t == 0 && bad) atomicAdd(&a.st->mismatch, 1);
    }
}

template <typename VT, int ACC, int ACC2>
hipError_t num_sg_impl(const NumArgs<VT> &a, const LaunchCfg &c) {
    int grid = c.grid;
    if (grid <= 0) grid = sg_resident_grid(ACC, ACC2, sizeof(VT) == 8, c.cus);
    if (a.b32) hipLaunchKernelGGL((k_num_sg<VT, ACC, ACC2, int32_t>), dim3(grid), dim3(SG_WG), 0, c.stream, a);
    else hipLaunchKernelGGL((k_num_sg<VT, ACC, ACC2, int64_t>), dim3(grid), dim3(SG_WG), 0, c.stream, a);
    return hipGetLastError();
}

}  // namespace

int sg_resident_grid(int acc, int acc2, bool dbl, int cus) {
    if (dbl) return resident_grid(k_num_sg<double, ACC_NATIVE, ACC_NATIVE, int64_t>, SG_WG, 0, cus);
    if (acc2 == ACC_WIDE && acc == ACC_NATIVE) return resident_grid(k_num_sg<float, ACC_NATIVE, ACC_WIDE, int64_t>, SG_WG, 0, cus);
    if (acc2 == ACC_WIDE && acc == ACC_COMP) return resident_grid(k_num_sg<float, ACC_COMP, ACC_WIDE, int64_t>, SG_WG, 0, cus);
    if (acc == ACC_COMP) return resident_grid(k_num_sg<float, ACC_COMP, ACC_COMP, int64_t>, SG_WG, 0, cus);
    if (acc == ACC_WIDE) return resident_grid(k_num_sg<float, ACC_WIDE, ACC_WIDE, int64_t>, SG_WG, 0, cus);
    return resident_grid(k_num_sg<float, ACC_NATIVE, ACC_NATIVE, int64_t>, SG_WG, 0, cus);
}

template <>
hipError_t launch_num_sg<double>(const NumArgs<double> &a, int, int, const LaunchCfg &c) {
    return num_sg_impl<double, ACC_NATIVE, ACC_NATIVE>(a, c);
}
template <>
hipError_t launch_num_sg<float>(const NumArgs<float> &a, int acc, int acc2, const LaunchCfg &c) {
    if (acc2 == ACC_WIDE && acc == ACC_NATIVE) return num_sg_impl<float, ACC_NATIVE, ACC_WIDE>(a, c);
    if (acc2 == ACC_WIDE && acc == ACC_COMP) return num_sg_impl<float, ACC_COMP, ACC_WIDE>(a, c);
    if (acc == ACC_COMP) return num_sg_impl<float, ACC_COMP, ACC_COMP>(a, c);
    if (acc == ACC_WIDE) return num_sg_impl<float, ACC_WIDE, ACC_WIDE>(a, c);
    return num_sg_impl<float, ACC_NATIVE, ACC_NATIVE>(a, c);
}

}  // namespace spg
