// Device helpers of the Legendre recurrence shared by the FP64 and the
// mixed-precision kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "sht_internal.h"

namespace sht {
namespace {

constexpr double kTwoS = 0x1p512;
constexpr double kTwoMinusS = 0x1p-512;

// mu * s^m as (v, k): value v 2^(512 k), k <= 0, v in (2^-513 mu, mu].
// Repeated squaring with the mantissa renormalised after every product.
__device__ inline void seed_mm(double mu, double s, int m, double &v, int &k)
{
    if (m == 0) { v = mu; k = 0; return; }
    if (s == 0.0) { v = 0.0; k = 0; return; }
    int e;
    double b = frexp(s, &e);
    int be = e;
    double r = 1.0;
    int re = 0;
    int p = m;
    while (p) {
        if (p & 1) {
            r *= b; re += be;
            r = frexp(r, &e); re += e;
        }
        p >>= 1;
        if (p) {
            b *= b; be *= 2;
            b = frexp(b, &e); be += e;
        }
    }
    int kk = (re < 0) ? -((-re) / kScaleStep) : 0;
    v = ldexp(mu * r, re - kScaleStep * kk);
    k = kk;
}

// Wave-uniform data that no kernel writes while it reads it comes through the
// constant address space: scalar loads, also where the compiler cannot prove
// that the kernel's stores leave it alone (the batch's workspace holds both
// the coefficients and Delta).
typedef const int __attribute__((address_space(4))) *CIp;
typedef const long long __attribute__((address_space(4))) *CLp;
typedef const double __attribute__((address_space(4))) *CDp;

// N doubles into scalar registers: vector-typed loads of 8-byte alignment, one
// s_load per 64 bytes.
typedef double d2a __attribute__((ext_vector_type(2), aligned(8)));
typedef double d4a __attribute__((ext_vector_type(4), aligned(8)));
typedef double d8a __attribute__((ext_vector_type(8), aligned(8)));

template <int N>
__device__ inline void scalar_rows(double *d, CDp p)
{
    if constexpr (N >= 8) {
        const d8a v = *(const d8a __attribute__((address_space(4))) *)p;
#pragma unroll
        for (int t = 0; t < 8; ++t) d[t] = v[t];
        if constexpr (N > 8) scalar_rows<N - 8>(d + 8, p + 8);
    } else if constexpr (N >= 4) {
        const d4a v = *(const d4a __attribute__((address_space(4))) *)p;
#pragma unroll
        for (int t = 0; t < 4; ++t) d[t] = v[t];
        if constexpr (N > 4) scalar_rows<N - 4>(d + 4, p + 4);
    } else {
        const d2a v = *(const d2a __attribute__((address_space(4))) *)p;
        d[0] = v[0];
        d[1] = v[1];
    }
}

// Waits for every scalar load on its way (they return out of order); nothing
// moves across.
__device__ inline void scalars_arrived()
{
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
    __builtin_amdgcn_sched_barrier(0);
}

}  // namespace
}  // namespace sht
