// Backward of C = A * B restricted to the stored entries of A and B.
//
// For L with dL/dC = G on pattern(C), each multiplication (i, k, j) of the
// numeric phase (A(i,k) and B(k,j) stored) contributes
//     dA(i,k) += G(i,j) * B(k,j)        dB(k,j) += A(i,k) * G(i,j)
// so dA = (G * B^T) masked to pattern(A) and dB = (A^T * G) masked to
// pattern(B).  One wavefront per row of A walks the row's multiplications
// flat, U per lane and round (neighbouring lanes on neighbouring B entries),
// finds G(i,j) by binary search in the sorted row i of C (columns and values
// staged in LDS when they fit), sums dA(i,k) over the lanes of a run by a
// segmented scan in FP64 and adds dB(k,j) with hardware atomics in HBM.
//
// Bound by the vector-memory path (its data unit 90% busy: a column and a value
// loaded and an atomic sent per product) with the VALU at 69%.  U searches per
// lane advance together, and LDS is sized by the longest row of C, so short rows
// leave room for 32 wavefronts per CU.  Backward of 7-point 64^3 times 16 random
// columns a row (2.9e7 multiplications, FP32): 273 us; with lane groups per B row, one search at a
// time and 16 KB of LDS per wavefront it took 1050 us.  (Sums over a run by LDS
// atomics would cost 190 cycles per 64 products: the lanes of a run share
// one address.)
#include "spg_accum.hpp"
#include "spg_flat.hpp"
#include "spg_internal.hpp"

namespace spg {

namespace {

constexpr int BW_LDS = 2048;  // entries of a C row staged in LDS (larger rows are searched in HBM)

// Value of the lane that a DPP move reads, 64-bit (0 where it reads none).
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_f64(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xF, false);
    return __hiloint2double(hi, lo);
}
// One step of the segmented inclusive scan: lanes of one run (equal k, never
// decreasing over the lanes) add the value the move brings.
template <int CTRL, int ROWS>
__device__ __forceinline__ void seg_step(double &v, int k) {
    const int ko = __builtin_amdgcn_update_dpp(-1, k, CTRL, ROWS, 0xF, false);
    const double vo = dpp_f64<CTRL, ROWS>(v);
    v += ko == k ? vo : 0.0;
}
__device__ __forceinline__ double seg_scan(double v, int k) {
    seg_step<0x111, 0xF>(v, k);  // row_shr:1
    seg_step<0x112, 0xF>(v, k);  // row_shr:2
    seg_step<0x114, 0xF>(v, k);  // row_shr:4
    seg_step<0x118, 0xF>(v, k);  // row_shr:8
    seg_step<0x142, 0xA>(v, k);  // row_bcast:15 into rows 1, 3
    seg_step<0x143, 0xC>(v, k);  // row_bcast:31 into rows 2, 3
    return v;
}

// rmax: entries of a C row that the dynamic LDS holds (power of two).
template <typename VT, typename IX, int U>
__global__ __launch_bounds__(WAVE) void k_bwd(BwdArgs<VT> a, int rmax) {
    extern __shared__ __align__(16) unsigned char smem[];
    VT *gval = (VT *)smem;
    int32_t *gcol = (int32_t *)(smem + sizeof(VT) * (size_t)rmax);
    __shared__ IX rel[WAVE], off[WAVE];  // per staged run (see spg_flat.hpp)
    __shared__ VT sav[WAVE];
    __shared__ double sdA[WAVE];
    __shared__ __align__(8) uint32_t wb[2 * U];
    const int l = lane_id();
    const Slice sl = xcd_slice(0, a.m);
    int64_t r = sl.idx;
    // software pipeline: the next row's first A entries, then their B row
    // extents, load during the current row
    int64_t ab = 0, ae = 0, nab = 0, nae = 0, b0 = 0, b1 = 0;
    VT av = VT(0);
    if (r < sl.end) {
        ab = a.arp[r];
        ae = a.arp[r + 1];
        if (ab + l < ae) {
            const int j = a.aci[ab + l];
            av = a.aval[ab + l];
            b0 = a.brp[j];
            b1 = a.brp[j + 1];
        }
    }
    if (r + sl.step < sl.end) {
        nab = a.arp[r + sl.step];
        nae = a.arp[r + sl.step + 1];
    }
    for (; r < sl.end; r += sl.step) {
        const int64_t cb = a.coff[r];
        const int rn = (int)(a.coff[r + 1] - cb);
        int lgr = 0;  // the search runs over 2^lgr - 1 entries or more, padded
        while ((1 << lgr) <= rn) ++lgr;
        const bool in_lds = (1 << lgr) <= rmax;
        int nj = 0;
        VT nav = VT(0);
        if (nab + l < nae) {
            nj = a.aci[nab + l];
            nav = a.aval[nab + l];
        }
        if (in_lds)
            for (int t = l; t < (1 << lgr); t += WAVE) {
                gcol[t] = t < rn ? a.gci[cb + t] : INT_MAX;
                gval[t] = t < rn ? a.gval[cb + t] : VT(0);
            }
        for (int64_t c0 = ab; c0 < ae; c0 += WAVE) {
            const int cn0 = (int)min((int64_t)WAVE, ae - c0);
            if (c0 != ab && l < cn0) {
                const int j = a.aci[c0 + l];
                av = a.aval[c0 + l];
                b0 = a.brp[j];
                b1 = a.brp[j + 1];
            }
            const long long len = l < cn0 ? b1 - b0 : 0;
            const long long inc = wave_incl_scan64(len + (len > 0 ? FLAT_ONE : 0));
            const long long all = __shfl(inc, WAVE - 1);
            const IX tot = (IX)(all & FLAT_LEN);
            const int cn = (int)(all >> FLAT_SHIFT), run = (int)(inc >> FLAT_SHIFT) - 1;
            wave_lds_sync();
            if (len > 0) {
                const long long end = inc & FLAT_LEN;
                off[run] = (IX)end;
                rel[run] = (IX)(b0 - (end - len));
                sav[run] = av;
            }
            sdA[l] = 0.0;
            wave_lds_sync();
            int kc = 0;
            for (IX F = 0; F < tot; F += (IX)(U * WAVE)) {
                int k[U], c[U], p[U];
                IX e[U];
                VT bv[U], gv[U];
                kc = flat_window<U>(off, cn, F, tot, kc, wb, k);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const IX f = F + (u * WAVE + l);
                    k[u] += kc;
                    e[u] = f < tot ? rel[k[u]] + f : IX(-1);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) c[u] = a.bci[e[u] < 0 ? 0 : e[u]];
#pragma unroll
                for (int u = 0; u < U; ++u) bv[u] = a.bval[e[u] < 0 ? 0 : e[u]];
                // entries of the row below column c, all U searches a step at a time
#pragma unroll
                for (int u = 0; u < U; ++u) p[u] = 0;
                if (in_lds) {
                    for (int s = (1 << lgr) >> 1; s > 0; s >>= 1)
#pragma unroll
                        for (int u = 0; u < U; ++u) p[u] += gcol[p[u] + s - 1] < c[u] ? s : 0;
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const bool hit = e[u] >= 0 && gcol[p[u]] == c[u];
                        gv[u] = gval[p[u]];
                        if (e[u] >= 0 && !hit) atomicAdd(&a.st->mismatch, 1);
                        if (!hit) e[u] = IX(-1);
                    }
                } else {
                    for (int s = (1 << lgr) >> 1; s > 0; s >>= 1)
#pragma unroll
                        for (int u = 0; u < U; ++u)
                            if (p[u] + s <= rn) p[u] += a.gci[cb + p[u] + s - 1] < c[u] ? s : 0;
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const bool hit = e[u] >= 0 && p[u] < rn && a.gci[cb + p[u]] == c[u];
                        gv[u] = hit ? a.gval[cb + p[u]] : VT(0);
                        if (e[u] >= 0 && !hit) atomicAdd(&a.st->mismatch, 1);
                        if (!hit) e[u] = IX(-1);
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (a.dB && e[u] >= 0) atomicAdd(&a.dB[e[u]], sav[k[u]] * gv[u]);
                    const double s = seg_scan(e[u] >= 0 ? (double)gv[u] * (double)bv[u] : 0.0, k[u]);
                    const int kn = __shfl_down(k[u], 1);
                    if (l == WAVE - 1 || kn != k[u]) atomicAdd(&sdA[k[u]], s);  // the last lane of each run
                }
            }
            wave_lds_sync();
            if (a.dA && l < cn0) a.dA[c0 + l] = len > 0 ? (VT)sdA[run] : VT(0);
        }
        ab = nab;
        ae = nae;
        av = nav;
        if (nab + l < nae) {
            b0 = a.brp[nj];
            b1 = a.brp[nj + 1];
        }
        if (r + 2 * sl.step < sl.end) {
            nab = a.arp[r + 2 * sl.step];
            nae = a.arp[r + 2 * sl.step + 1];
        } else {
            nab = nae = 0;
        }
        wave_lds_sync();
    }
}

template <typename VT>
__global__ void k_zero(VT *p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = VT(0);
}

template <typename VT, typename IX, int U>
hipError_t bwd_launch(const BwdArgs<VT> &a, const LaunchCfg &c) {
    int rmax = WAVE;
    while (rmax <= a.max_row && rmax < BW_LDS) rmax <<= 1;
    const size_t lds = (4 + sizeof(VT)) * (size_t)rmax;
    const int grid = resident_grid(k_bwd<VT, IX, U>, WAVE, lds, c.cus);
    hipLaunchKernelGGL((k_bwd<VT, IX, U>), dim3(grid), dim3(WAVE), lds, c.stream, a, rmax);
    return hipGetLastError();
}

// U = 2 for rows of up to 2 * 64 multiplications on average (a row's products
// then fill a round), else 8; 32-bit product numbers where 64 A entries cannot
// form 2^31 products.
template <typename VT>
hipError_t bwd_impl(const BwdArgs<VT> &a, const LaunchCfg &c) {
    if (a.dB && a.nnzb > 0) {
        const int64_t blocks = std::min<int64_t>((a.nnzb + 255) / 256, 8192);
        hipLaunchKernelGGL(k_zero<VT>, dim3((unsigned)blocks), dim3(256), 0, c.stream, a.dB, a.nnzb);
    }
    if (a.m == 0) return hipGetLastError();
    const bool i32 = flat_32bit(a.nnzb, WAVE, 8 * WAVE);
    if (a.flops <= 2 * WAVE * a.m)
        return i32 ? bwd_launch<VT, int32_t, 2>(a, c) : bwd_launch<VT, int64_t, 2>(a, c);
    return i32 ? bwd_launch<VT, int32_t, 8>(a, c) : bwd_launch<VT, int64_t, 8>(a, c);
}

}  // namespace

template <>
hipError_t launch_backward<double>(const BwdArgs<double> &a, const LaunchCfg &c) {
    return bwd_impl<double>(a, c);
}
template <>
hipError_t launch_backward<float>(const BwdArgs<float> &a, const LaunchCfg &c) {
    return bwd_impl<float>(a, c);
}

}  // namespace spg
