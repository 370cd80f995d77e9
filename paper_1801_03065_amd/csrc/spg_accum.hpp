// Accumulator arithmetic shared by the numeric kernels.
//
// Three forms of "C(i,j) += A(i,k) * B(k,j)":
//   ACC_NATIVE: product and sum in the value type (FP64 for the plain method,
//               FP32 for the single-precision form); FP64 and HBM sums by
//               hardware atomic add, FP32 sums in LDS by lds_add_f32.
//   ACC_COMP:   FP32 values, compensated pair (s, c) per entry: TwoProduct of
//               the operands (exact error by fused multiply-add), TwoSum into s,
//               both errors into c; the pair is one 64-bit word updated by
//               compare-and-swap.  Result s + c (Ogita, Rump, Oishi, "Accurate
//               sum and dot product", 2005, algorithm Dot2).
//   ACC_WIDE:   FP32 values, FP64 accumulation (the product of two FP32 numbers
//               is exact in FP64).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace spg {

enum { ACC_NATIVE = 0, ACC_COMP = 1, ACC_WIDE = 2 };

// *p += x for FP32 accumulators in LDS.  The LDS unit serialises ds_add_f32
// over the lanes: 193 cycles of a CU per 64-lane instruction whatever the
// addresses, against 12-22 for ds_add_f64 and 18-28 for a read and a
// compare-and-swap (measured with 16 wavefronts per CU on 256 to 1024
// addresses).  So the sum goes by compare-and-swap; each try serves one lane
// per address, and lanes that lost F32_TRIES of them (many lanes on one
// address) take the atomic add, whose cost is that of the lanes left.
// 27-point A*A on 61^3, FP32 numeric: 905 -> 329 us.
constexpr int F32_TRIES = 6;
__device__ __forceinline__ void lds_add_f32(float *p, float x) {
    // the address space is named: inside the loop the compiler loses it
    typedef __attribute__((address_space(3))) uint32_t lds_u32;
    typedef __attribute__((address_space(3))) float lds_f32;
    lds_u32 *u = (lds_u32 *)(uint32_t *)p;
    uint32_t old = __hip_atomic_load(u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    for (int k = 0; k < F32_TRIES; ++k) {
        const uint32_t sum = __float_as_uint(__uint_as_float(old) + x);
        if (__hip_atomic_compare_exchange_strong(u, &old, sum, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_WORKGROUP))
            return;
    }
    __hip_atomic_fetch_add((lds_f32 *)p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// add: accumulators in LDS; add_hbm: accumulators in HBM.
template <typename VT, int ACC>
struct Accum;

template <>
struct Accum<double, ACC_NATIVE> {
    using store_t = double;
    static __device__ __forceinline__ void add(store_t *p, double a, double b) { atomicAdd(p, a * b); }
    static __device__ __forceinline__ void add_hbm(store_t *p, double a, double b) { atomicAdd(p, a * b); }
    static __device__ __forceinline__ double fin(store_t v) { return v; }
    static __device__ __forceinline__ store_t zero() { return 0.0; }
};

template <>
struct Accum<float, ACC_NATIVE> {
    using store_t = float;
    static __device__ __forceinline__ void add(store_t *p, float a, float b) { lds_add_f32(p, a * b); }
    static __device__ __forceinline__ void add_hbm(store_t *p, float a, float b) { atomicAdd(p, a * b); }
    static __device__ __forceinline__ float fin(store_t v) { return v; }
    static __device__ __forceinline__ store_t zero() { return 0.0f; }
};

template <>
struct Accum<float, ACC_WIDE> {
    using store_t = double;
    static __device__ __forceinline__ void add(store_t *p, float a, float b) {
        atomicAdd(p, (double)a * (double)b);
    }
    static __device__ __forceinline__ void add_hbm(store_t *p, float a, float b) { add(p, a, b); }
    static __device__ __forceinline__ float fin(store_t v) { return (float)v; }
    static __device__ __forceinline__ store_t zero() { return 0.0; }
};

template <>
struct Accum<float, ACC_COMP> {
    using store_t = unsigned long long;  // low word s, high word c
    static __device__ __forceinline__ void add(store_t *p, float a, float b) {
        const float x = a * b;
        const float ex = __builtin_fmaf(a, b, -x);  // a*b == x + ex exactly
        store_t old = *(volatile store_t *)p, assumed;
        do {
            assumed = old;
            const float s = __uint_as_float((uint32_t)assumed);
            const float c = __uint_as_float((uint32_t)(assumed >> 32));
            const float s2 = s + x;  // TwoSum(s, x) = (s2, e), s + x == s2 + e exactly
            const float bv = s2 - s;
            const float e = (s - (s2 - bv)) + (x - bv);
            const float c2 = c + (e + ex);
            const store_t nv = (store_t)__float_as_uint(s2) | ((store_t)__float_as_uint(c2) << 32);
            old = atomicCAS(p, assumed, nv);
        } while (old != assumed);
    }
    static __device__ __forceinline__ void add_hbm(store_t *p, float a, float b) { add(p, a, b); }
    static __device__ __forceinline__ float fin(store_t v) {
        return __uint_as_float((uint32_t)v) + __uint_as_float((uint32_t)(v >> 32));
    }
    static __device__ __forceinline__ store_t zero() { return 0ull; }
};

__host__ __device__ constexpr size_t align16(size_t x) { return (x + 15) & ~size_t(15); }

// A product as it is kept until its run is summed, and the sum of a run.
// FP64: the product.  FP32 plain: the product rounded to FP32, FP32 sums.
// FP32 compensated and FP64-accumulated: the exact product in FP64; the
// compensated pair takes its FP32 rounding and the error from it.
template <typename VT, int ACC>
struct BkTerm {
    using term_t = typename std::conditional<ACC == ACC_NATIVE, VT, double>::type;
    static __device__ __forceinline__ term_t term(VT a, VT b) { return (term_t)a * (term_t)b; }
    term_t s = term_t(0);
    __device__ __forceinline__ void add(term_t x) { s += x; }
    __device__ __forceinline__ VT fin() const { return (VT)s; }
};
template <>
struct BkTerm<float, ACC_COMP> {
    using term_t = double;
    static __device__ __forceinline__ double term(float a, float b) { return (double)a * (double)b; }
    float s = 0.0f, c = 0.0f;
    __device__ __forceinline__ void add(double p) {
        const float x = (float)p, ex = (float)(p - (double)x);  // p == x + ex exactly
        const float s2 = s + x, bv = s2 - s;                     // TwoSum(s, x)
        c += ((s - (s2 - bv)) + (x - bv)) + ex;
        s = s2;
    }
    __device__ __forceinline__ float fin() const { return s + c; }
};

}  // namespace spg
