// Pieces shared by the mixed-precision Legendre kernels: the lanes' recurrence,
// and, for the two split forms, the exchange of fragment halves, the output
// tiles and the Delta epilogue.
#pragma once

#include "recurrence.h"
#include "sht_internal.h"

namespace sht {
namespace {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef unsigned int v2u __attribute__((ext_vector_type(2)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));

__device__ inline void swap_halves(float a, float b, float &lo, float &hi)
{
    const v2u r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b),
                                                   false, false);
    lo = __uint_as_float(r[0]);
    hi = __uint_as_float(r[1]);
}

struct MfmaTiles {
    v16f e0, e1, o0, o1;  // even / odd parity, rows 0-31 / 32-63
};

__device__ __forceinline__ void zero_tiles(MfmaTiles &t)
{
    t.e0 = v16f{}; t.e1 = v16f{}; t.o0 = v16f{}; t.o1 = v16f{};
}

__device__ __forceinline__ void add_tiles(MfmaTiles &tot, const MfmaTiles &acc)
{
    tot.e0 += acc.e0; tot.e1 += acc.e1; tot.o0 += acc.o0; tot.o1 += acc.o1;
}

// Waves to a workgroup.  They share nothing, and one each suits most launches (a
// wave that is done makes room for the next; up to three to a CU have a SIMD
// each).  With about one to a SIMD single waves land unevenly on the SIMDs, and
// four to a workgroup take less time (Legendre stage of 16 maps and 64 m at
// l_max 2048 / nside 1024, 1024 waves: FP32 435 and 327 us, FP16x2 210 and 174,
// BF16x3 277 and 239; with 768 waves 283 and 289, 140 and 143, 204 and 209; with
// 1280 482 and 493, 258 and 259, 318 and 332).
inline int waves_per_group(const sht_plan_s *p, long long waves)
{
    return waves > 3LL * p->num_cus && 2 * waves <= 9LL * p->num_cus ? 4 : 1;
}

// This wave's place in an XCD's list of waves (workgroups are dealt to the 8
// XCDs round-robin).
template <int W>
__device__ __forceinline__ int xcd_wave()
{
    // uniform over the wave
    return (int)(blockIdx.x / 8) * W +
           (W > 1 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) : 0);
}

// A lane's recurrence on one m: zero until its start row, where it takes the
// start table's values (`stash`, its LDS slot).  Before it the true values are
// below 2^-160, which is zero in FP32, so a lane's operands need no mask, and
// from there on they are plain FP64 values bounded by sqrt((2l+1)/4pi)/c_l <
// 2^9 (addition theorem).
struct Lane {
    double x, ua, ub;
    int je;              // start row, units of kLiveRows
};

// 8 rows from row r on (coefficients a), as FP32 values of both parities.
__device__ __forceinline__ void rows8(Lane &l, const double *a, float *ve, float *vo)
{
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const double u0 = fma(a[2 * t] * l.x, l.ub, -l.ua);
        const double u1 = fma(a[2 * t + 1] * l.x, u0, -l.ub);
        l.ua = u0;
        l.ub = u1;
        ve[t] = (float)u0;
        vo[t] = (float)u1;
    }
}

// Lanes that start at row r take their values, times `scale`.  `last`: no
// lane of the wave starts after it (uniform).
__device__ __forceinline__ void enter(Lane &l, const double2 *stash, int r, int last,
                                      double scale = 1.0)
{
    if (r <= last) {
        asm volatile("");   // a branch of its own, around the lane compare too
        if (l.je == r / kLiveRows) {
            const double2 v = *stash;
            l.ua = v.x * scale;
            l.ub = v.y * scale;
        }
    }
}

// Delta of one m.  D layout of a 32x32 tile: column = lane % 32 (the ring
// pair), row = 8 (r/4) + 4 (lane/32) + r % 4 = 2 map + Re/Im, so a lane owns
// 8 complex values of one pair.  The mixed forms' Delta has the maps
// of a ring contiguous: the ring stage reads a ring's modes for all maps at
// once, and the wave writes every map of its rings, so each line is filled
// by one wave.  The parity sums are FP32; north (E + O) and south (E - O)
// are formed exactly in FP64 and rounded once to FP32, the precision the
// contraction carries, so Delta is stored as complex64.
__device__ __forceinline__ void m_store(const MfmaTiles &tot, int i, float2 *__restrict__ delta,
                                        const PairDesc *__restrict__ pairs, int npairs, int pb,
                                        int grp, int nmaps, const DeltaLayout &dl, bool full,
                                        int lane)
{
    const int hi = lane >> 5;
    const int col = lane & 31;
    float2 *__restrict__ d2 = delta;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const v16f &E = h ? tot.e1 : tot.e0;
        const v16f &O = h ? tot.o1 : tot.o0;
        const int pp = pb * 64 + h * 32 + col;
        if (pp < npairs) {
            const PairDesc d = pairs[pp];
            if (!full && i >= d.ilim32) continue;   // dead on the ring, not read
            const int rs = d.rs >= 0 ? d.rs : d.rn;
            float2 *__restrict__ dn = d2 + dl.row(d.rn) + i * dl.mstride(d.rn);
            float2 *__restrict__ ds = d2 + dl.row(rs) + i * dl.mstride(rs);
#pragma unroll
            for (int r = 0; r < 16; r += 4) {
                // rows r .. r + 3: maps m0 and m0 + 1, adjacent in Delta, so
                // one 16-byte store takes both when the alignment allows
                const int m0 = grp * 16 + 4 * (r >> 2) + 2 * hi;
                float2 n[2], so[2];
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const double er = E[r + 2 * k], ei = E[r + 2 * k + 1];
                    const double orr = O[r + 2 * k], oi = O[r + 2 * k + 1];
                    n[k] = make_float2((float)(er + orr), (float)(ei + oi));
                    so[k] = make_float2((float)(er - orr), (float)(ei - oi));
                }
                if (m0 + 1 < nmaps && (nmaps & 1) == 0) {
                    *reinterpret_cast<float4 *>(dn + m0) =
                        make_float4(n[0].x, n[0].y, n[1].x, n[1].y);
                    if (d.rs >= 0)
                        *reinterpret_cast<float4 *>(ds + m0) =
                            make_float4(so[0].x, so[0].y, so[1].x, so[1].y);
                } else {
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        if (m0 + k < nmaps) {
                            dn[m0 + k] = n[k];
                            if (d.rs >= 0) ds[m0 + k] = so[k];
                        }
                    }
                }
            }
        }
    }
}

}  // namespace
}  // namespace sht
