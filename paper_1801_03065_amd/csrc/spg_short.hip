// Short rows: several rows of C per wavefront (Partitioning Schemes
// subsection, Thread-Parallel with a team of lanes per row).
//
// A row whose multiplication count f_m(i) is at most T = 2^lg_t lanes is
// handled by a team of T lanes, WAVE / T rows at once.  The row's products
// are spread one per lane (expansion: prefix sum of the B row lengths over
// the row of A, then each lane counts the B rows that start up to it).
//   symbolic: the columns go into a team-private linear-probing hash in LDS
//             (LP hashmap, Accumulators subsection: 2T slots, so at most 50%
//             occupancy); row size = number of first insertions.
//   numeric:  (column, lane) is sorted across the team with a bitonic network
//             on one 32-bit key; equal columns are neighbours then, in product
//             order, and the first of each run adds the others' products.
// The per-row cost of a whole wavefront (stage, scans, summary) is what this
// avoids: for rows of a few dozen multiplications it dominates.  Like the
// wavefront kernels, the loop is software-pipelined across rows: the next
// row's A entries and B extents load while the current row is processed.
//
// Bound by random lines of B past the L2 where B is large (1.5M rows of 7
// random entries: 5.1 TB/s symbolic, 6.2 numeric), else by the vector-memory data
// unit (Galerkin products on 100^3: 82 to 93% busy).  Numeric, the same
// product: 1032 us with a hash of the products, sorted (column, slot) pairs
// after it; 665 us now.  Galerkin products on 100^3, both: 394 -> 343 us; 7-point
// 100^3: 699 -> 606 us.  (Symbolic, sorting took 428 us and the hash 379.)
#include "spg_accum.hpp"
#include "spg_internal.hpp"

namespace spg {

namespace {

template <typename VT>
struct SrArgs {
    const int64_t *arp;
    const int32_t *aci;
    const VT *aval;  // numeric only
    const int64_t *brp;
    const int32_t *bci;
    const VT *bval;  // numeric only
    const int64_t *coff;
    int32_t *cci;
    VT *cval;
    int64_t cbase_row;
    int32_t *row_nnz;    // symbolic only
    int32_t *row_words;  // symbolic only (row size as the word bound)
    RowSet rs;
    DevStats *st;
};

// Value of lane (lane ^ J): DPP quad permutes for 1 and 2, a row rotation
// for 8, swizzles inside 32 lanes for 4 and 16, a lane permute for 32.
template <int J>
__device__ __forceinline__ int lane_xor(int v) {
    if (J == 1) return __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, false);   // quad_perm [1,0,3,2]
    if (J == 2) return __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, false);   // quad_perm [2,3,0,1]
    if (J == 8) return __builtin_amdgcn_mov_dpp(v, 0x128, 0xF, 0xF, false);  // row_ror:8
    if (J == 4) return __builtin_amdgcn_ds_swizzle(v, 0x1F | (4 << 10));
    if (J == 16) return __builtin_amdgcn_ds_swizzle(v, 0x1F | (16 << 10));
    return __shfl_xor(v, J);
}
// Slot of column c in a table of 2^lg slots (Fibonacci hash of the low 24 bits).
__device__ __forceinline__ uint32_t sr_hash(int c, int lg) {
    return (__umul24((uint32_t)c & 0xFFFFFFu, 0x9E3779u) >> (24 - lg)) & ((1u << lg) - 1u);
}
// One compare-exchange step of the bitonic network (block size KK, distance J).
template <int KK, int J>
__device__ __forceinline__ void bitonic_step(uint32_t &key, int q) {
    const uint32_t ok = (uint32_t)lane_xor<J>((int)key);
    const bool up = (q & KK) == 0, lower = (q & J) == 0;
    key = lower == up ? min(key, ok) : max(key, ok);
}
template <int KK, int J>
__device__ __forceinline__ void bitonic_step(uint64_t &key, int q) {
    const uint32_t ol = (uint32_t)lane_xor<J>((int)(uint32_t)key), oh = (uint32_t)lane_xor<J>((int)(uint32_t)(key >> 32));
    const uint64_t ok = (uint64_t)oh << 32 | ol;
    const bool up = (q & KK) == 0, lower = (q & J) == 0;
    if (lower == up ? ok < key : ok > key) key = ok;
}
// Sort ascending inside blocks of P lanes (P <= 2^LG, a power of two,
// wavefront-uniform): the stages for blocks above P are skipped.
template <int LG, typename KEY>
__device__ __forceinline__ void team_sort(KEY &key, int q, int P) {
#define SR_STAGE(KK, J) bitonic_step<KK, J>(key, q);
    SR_STAGE(2, 1)
    if (P < 4) return;
    SR_STAGE(4, 2) SR_STAGE(4, 1)
    if (P < 8) return;
    SR_STAGE(8, 4) SR_STAGE(8, 2) SR_STAGE(8, 1)
    if (LG < 4 || P < 16) return;
    SR_STAGE(16, 8) SR_STAGE(16, 4) SR_STAGE(16, 2) SR_STAGE(16, 1)
    if (LG < 5 || P < 32) return;
    SR_STAGE(32, 16) SR_STAGE(32, 8) SR_STAGE(32, 4) SR_STAGE(32, 2) SR_STAGE(32, 1)
    if (LG < 6 || P < 64) return;
    SR_STAGE(64, 32) SR_STAGE(64, 16) SR_STAGE(64, 8) SR_STAGE(64, 4) SR_STAGE(64, 2) SR_STAGE(64, 1)
#undef SR_STAGE
}

// Largest value (>= 0) of the 64 lanes, uniform.
__device__ __forceinline__ int sr_wave_max(int v) {
    return __builtin_amdgcn_readlane(wave_maxscan_dpp(v), WAVE - 1);
}
// Value of the team's last lane.
template <int LG>
__device__ __forceinline__ int team_last(int v) {
    if (LG == 6) return __builtin_amdgcn_readlane(v, WAVE - 1);
    return __shfl(v, (1 << LG) - 1, 1 << LG);
}

// NUM: values (else the row's distinct columns are counted).  PACK: columns
// below 2^26 and 32-bit byte offsets into B: (column, lane) fits 32 bits.
template <bool NUM, typename VT, int ACC, int LG, bool PACK>
__global__ __launch_bounds__(WAVE) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_sr(SrArgs<VT> a) {
    using Term = BkTerm<VT, ACC>;
    using P = typename Term::term_t;
    using IX = typename std::conditional<PACK, int32_t, int64_t>::type;
    using KEY = typename std::conditional<PACK, uint32_t, uint64_t>::type;  // column, lane
    __shared__ __align__(8) uint32_t starts[2];  // wavefront lanes where a B row's products start
    __shared__ IX rel[WAVE];                     // per nonempty B row: its start less its first product's lane
    __shared__ VT sav[NUM ? WAVE : 1];
    __shared__ P vals[NUM ? WAVE : 1];
    __shared__ int32_t keys[NUM ? 1 : 2 * WAVE];  // hash of 2T slots per team
    const int l = lane_id();
    constexpr int T = 1 << LG;
    const int q = l & (T - 1), team = l >> LG;
    constexpr int nteam = WAVE >> LG;
    const unsigned long long below = team ? (1ull << (team * T)) - 1 : 0ull;  // lanes of the teams before
    const unsigned long long mine_m = (T == 64 ? ~0ull : ((1ull << (T & 63)) - 1) << (team * T & 63));
    if (!NUM) {
        keys[l] = -1;
        keys[l + WAVE] = -1;
        wave_lds_sync();
    }
    int64_t lo, hi;
    rs_bounds(a.rs, lo, hi);
    const int64_t ngroups = (hi - lo + nteam - 1) / nteam;
    const Slice sl = xcd_slice(0, ngroups);
    const int64_t cbase = (NUM && a.cbase_row >= 0) ? a.coff[a.cbase_row] : 0;

    // this team's row in group gg, or -1
    auto row_of = [&](int64_t gg) -> int {
        const int64_t r = lo + gg * nteam + team;
        return (gg < sl.end && r < hi) ? a.rs.rows[r] : -1;
    };

    int64_t g = sl.idx;
    int ic = row_of(g);
    int64_t abc = 0, aec = 0;
    if (ic >= 0) {
        abc = a.arp[ic];
        aec = a.arp[ic + 1];
    }
    int lenc = 0;
    int64_t b0c = 0;
    VT avc = VT(0);
    if (q < aec - abc) {
        const int j = a.aci[abc + q];
        if (NUM) avc = a.aval[abc + q];
        b0c = a.brp[j];
        lenc = (int)(a.brp[j + 1] - b0c);
    }
    int in = row_of(g + sl.step);
    int64_t abn = 0, aen = 0;
    if (in >= 0) {
        abn = a.arp[in];
        aen = a.arp[in + 1];
    }
    int i2 = row_of(g + 2 * sl.step);  // row indices load two groups ahead
    while (g < sl.end) {
        // next row, first level: its A entries (first chunk)
        int jn = 0;
        VT avn = VT(0);
        if (q < aen - abn) {
            jn = a.aci[abn + q];
            if (NUM) avn = a.aval[abn + q];
        }
        int64_t cb = 0, ce = 0;
        if (NUM && ic >= 0) {
            cb = a.coff[ic];
            ce = a.coff[ic + 1];
        }
        // ---- one product per lane
        IX e = 0;
        VT avk = avc;
        bool mine;
        int F, span;  // the team's products; lanes they lie in
        const bool more = __ballot(aec - abc > T) != 0;  // A rows with empty B rows, in chunks of T entries
        if (!more && __ballot(lenc > 1) == 0) {
            // B rows of at most one entry (every A entry makes at most one
            // product, e.g. aggregation or injection operators): each lane
            // forms its own product, no expansion
            e = (IX)b0c;
            mine = lenc > 0;
            F = __popcll(__ballot(mine) & mine_m);
            span = (int)(aec - abc);
        } else {
            F = 0;
            mine = false;
            int len = lenc;
            int64_t b0 = b0c;
            VT av = avc;
            for (int64_t c0 = 0;;) {  // the same number of chunks in every team
                const int inc = team_scan<LG>(len, q), off = F + inc - len;
                const int Fc = team_last<LG>(inc);
                const unsigned long long runs = __ballot(len > 0 && off < T);
                if (l < 2) starts[l] = 0u;
                wave_lds_sync();
                if (len > 0 && off < T) {
                    const int at = team * T + off, run = mbcnt(runs);
                    atomicOr(&starts[at >> 5], 1u << (at & 31));
                    rel[run] = (IX)(b0 - at);
                    if (NUM) sav[run] = av;
                }
                wave_lds_sync();
                const uint32_t s0 = read_first((int)starts[0]), s1 = read_first((int)starts[1]);
                // a lane's run: the starts up to it, less one
                const int k = __builtin_amdgcn_mbcnt_hi(s1 >> 1, __builtin_amdgcn_mbcnt_lo(s0 >> 1 | s1 << 31, (s0 & 1) - 1));
                if (q >= F && q < F + Fc) {
                    e = rel[max(k, 0)] + l;
                    if (NUM) avk = sav[max(k, 0)];
                    mine = true;
                }
                F += Fc;
                c0 += T;
                if (!more || __ballot(abc + c0 < aec) == 0) break;
                len = 0;
                if (abc + c0 + q < aec) {
                    const int j = a.aci[abc + c0 + q];
                    if (NUM) av = a.aval[abc + c0 + q];
                    b0 = a.brp[j];
                    len = (int)(a.brp[j + 1] - b0);
                }
                wave_lds_sync();
            }
            if (q == 0 && F > T) atomicAdd(&a.st->mismatch, 1);  // not a short row: plan inconsistent
            F = min(F, T);
            span = F;
        }
        if constexpr (!NUM) {  // distinct columns: first insertions
            int fresh = 0;
            if (mine) {
                const int col = PACK ? ld32(a.bci, (uint32_t)e) : a.bci[e];
                uint32_t h = sr_hash(col, LG + 1);
                for (;;) {
                    const int old = atomicCAS(&keys[2 * T * team + h], -1, col);
                    fresh = old == -1;
                    if (fresh || old == col) break;
                    h = (h + 1) & (2u * T - 1u);
                }
            }
            const int cnt = __popcll(__ballot(fresh) & mine_m);
            if (q == 0 && ic >= 0) {
                a.row_nnz[ic] = cnt;
                a.row_words[ic] = cnt;
            }
            wave_lds_sync();
            keys[l] = -1;
            keys[l + WAVE] = -1;
        } else {
            KEY key = ~(KEY)0;
            if (mine) {
                const int col = PACK ? ld32(a.bci, (uint32_t)e) : a.bci[e];
                const VT bv = PACK ? ld32(a.bval, (uint32_t)e) : a.bval[e];
                vals[l] = Term::term(avk, bv);
                key = (KEY)(uint32_t)col << 6 | l;
            }
            // ---- sorted by column over the next power of two of the wavefront's
            // largest row; equal columns are neighbours then, in product order
            {
                const int mc = LG == 6 ? read_first(span) : sr_wave_max(span);
                int p2 = 2;
                while (p2 < mc) p2 <<= 1;
                team_sort<LG>(key, q, p2);
            }
            const int col = (int)(uint32_t)(key >> 6);
            const int pcol = __shfl_up(col, 1);
            const bool head = q < F && (q == 0 || col != pcol);
            const unsigned long long hm = __ballot(head);
            const int cnt = __popcll(hm & mine_m);
            wave_lds_sync();
            const P v = vals[(uint32_t)key & 63u];
            Term s;
            s.add(v);
            if (__ballot(q < F && !head)) {  // repeated columns: a head adds the products up to the next one
                wave_lds_sync();
                vals[l] = v;
                wave_lds_sync();
                const unsigned long long rest = hm >> l >> 1;
                const int next = min(rest ? l + 1 + (__ffsll((long long)rest) - 1) : WAVE, team * T + F);
                const int run = head ? next - l : 0, longest = sr_wave_max(run);
                for (int x = 1; x < longest; ++x)
                    if (x < run) s.add(vals[l + x]);
            }
            const bool okrow = ic < 0 || ce - cb == cnt;
            if (q == 0 && !okrow) atomicAdd(&a.st->mismatch, 1);
            if (okrow && head) {
                const int64_t o = cb - cbase + (mbcnt(hm) - __popcll(hm & below));
                a.cci[o] = col;
                a.cval[o] = s.fin();
            }
        }
        // next row, second level: B extents of its first chunk
        int64_t b0n = 0;
        int lenn = 0;
        if (q < aen - abn) {
            b0n = a.brp[jn];
            lenn = (int)(a.brp[jn + 1] - b0n);
        }
        // the row after next: its A extent (its index loaded a group ago)
        g += sl.step;
        const int inn = i2;
        int64_t abnn = 0, aenn = 0;
        if (inn >= 0) {
            abnn = a.arp[inn];
            aenn = a.arp[inn + 1];
        }
        i2 = row_of(g + 2 * sl.step);
        ic = in;
        abc = abn;
        aec = aen;
        avc = avn;
        b0c = b0n;
        lenc = lenn;
        in = inn;
        abn = abnn;
        aen = aenn;
        wave_lds_sync();
    }
}

template <bool NUM, typename VT, int ACC, int LG, bool PACK>
hipError_t sr_pack(const SrArgs<VT> &a, const LaunchCfg &c, int64_t rows) {
    const int64_t groups = (rows >> (6 - LG)) + XCDS - 1;
    const int grid = c.grid > 0 ? c.grid : (int)std::min<int64_t>(resident_grid(k_sr<NUM, VT, ACC, LG, PACK>, WAVE, 0, c.cus),
                                                                  std::max<int64_t>(XCDS, groups / XCDS * XCDS));
    hipLaunchKernelGGL((k_sr<NUM, VT, ACC, LG, PACK>), dim3(grid), dim3(WAVE), 0, c.stream, a);
    return hipGetLastError();
}
template <typename VT, int ACC, int LG>
hipError_t num_sr_lg(const SrArgs<VT> &a, bool pack, const LaunchCfg &c, int64_t rows) {
    return pack ? sr_pack<true, VT, ACC, LG, true>(a, c, rows) : sr_pack<true, VT, ACC, LG, false>(a, c, rows);
}

template <typename VT, int ACC>
hipError_t num_sr_impl(const NumArgs<VT> &n, int lg_t, const LaunchCfg &c, int64_t rows) {
    SrArgs<VT> a{};
    a.arp = n.arp;
    a.aci = n.aci;
    a.aval = n.aval;
    a.brp = n.brp;
    a.bci = n.bci;
    a.bval = n.bval;
    a.coff = n.coff;
    a.cci = n.cci;
    a.cval = n.cval;
    a.cbase_row = n.cbase_row;
    a.rs = n.rs;
    a.st = n.st;
    const bool pack = n.b32 && n.ncols <= (int64_t(1) << 26);
    if (lg_t <= 3) return num_sr_lg<VT, ACC, 3>(a, pack, c, rows);
    if (lg_t == 4) return num_sr_lg<VT, ACC, 4>(a, pack, c, rows);
    if (lg_t == 5) return num_sr_lg<VT, ACC, 5>(a, pack, c, rows);
    return num_sr_lg<VT, ACC, 6>(a, pack, c, rows);
}

template <int LG>
hipError_t sym_sr_lg(const SrArgs<double> &a, bool b32, const LaunchCfg &c, int64_t rows) {
    return b32 ? sr_pack<false, double, ACC_NATIVE, LG, true>(a, c, rows)
               : sr_pack<false, double, ACC_NATIVE, LG, false>(a, c, rows);
}

}  // namespace

hipError_t launch_sym_sr(const SymArgs &s, int lg_t, const LaunchCfg &c, int64_t rows) {
    if (lg_t < 0 || lg_t > 6) return hipErrorInvalidValue;
    SrArgs<double> a{};
    a.arp = s.arp;
    a.aci = s.aci;
    a.brp = s.brp;
    a.bci = s.bci;
    a.row_nnz = s.row_nnz;
    a.row_words = s.row_words;
    a.rs = s.rs;
    a.st = s.st;
    a.cbase_row = -1;
    if (lg_t <= 3) return sym_sr_lg<3>(a, s.b32, c, rows);
    if (lg_t == 4) return sym_sr_lg<4>(a, s.b32, c, rows);
    if (lg_t == 5) return sym_sr_lg<5>(a, s.b32, c, rows);
    return sym_sr_lg<6>(a, s.b32, c, rows);
}

template <>
hipError_t launch_num_sr<double>(const NumArgs<double> &a, int, int lg_t, const LaunchCfg &c, int64_t rows) {
    if (lg_t < 0 || lg_t > 6) return hipErrorInvalidValue;
    return num_sr_impl<double, ACC_NATIVE>(a, lg_t, c, rows);
}
template <>
hipError_t launch_num_sr<float>(const NumArgs<float> &a, int acc, int lg_t, const LaunchCfg &c, int64_t rows) {
    if (lg_t < 0 || lg_t > 6) return hipErrorInvalidValue;
    if (acc == ACC_COMP) return num_sr_impl<float, ACC_COMP>(a, lg_t, c, rows);
    if (acc == ACC_WIDE) return num_sr_impl<float, ACC_WIDE>(a, lg_t, c, rows);
    return num_sr_impl<float, ACC_NATIVE>(a, lg_t, c, rows);
}

}  // namespace spg
