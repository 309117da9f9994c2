// Start tables of the Legendre recurrence (plan time).
//
// P_mm = mu_m sin^m(theta) lies far below the smallest double for most
// (m, ring): the functions of an m stay negligible up to l ~ m / sin(theta),
// then grow within a few dozen steps to order one (Sec. 2.2.2 rescales the
// recurrence through that range at run time).  Where they start to count does
// not depend on the coefficients, so the plan finds it once: for every
// (m, ring pair) the first row j = l - m, in units of kLiveRows, from which
// the values pass a floor, and the two recurrence values there.  The
// transforms begin at that row, from true FP64 values: no rescaling, and
// nothing at all for the (m, ring) with no live row.
//
// The floor of the FP64 kernels is 2^-960.  A floor relative to what an m
// reaches later (2^-192 of it, say) would save more, but a Delta or a
// coefficient may consist of just those small terms: one coefficient near
// l = m, a spectrum that falls by more than 2^130 within an m (smoothing by
// a wide beam), rings near a pole alone.  Down to 2^-960 every term counts to
// full precision: a value grows by less than 2^55 over the 8 rows of a block
// (l <= 16383), so the value before a start row is a normal number, and
// the one before that, at most two steps of 2^7 smaller, enters the next with
// a weight of 2^-14.
//
// The mixed forms' Legendre kernels round P_lm to FP32 (or less), where
// everything below 2^-150 is zero: their table has a floor of 2^-160.  Their
// plans have both, since the adjoint is FP64.
//
// Of the (l, m, ring) terms at l_max 4096 / nside 2048 17% lie below 2^-960 and
// 28% below 2^-160 (l_max 1024: 6 and 20%).  A table takes 18 bytes per (m,
// pair), 0.6 of a map's complex128 Delta.
#include "recurrence.h"
#include "sht_internal.h"

namespace sht {
namespace {

constexpr double kFloor64 = 0x1p-960;
constexpr double kFloor32 = 0x1p-160;
constexpr double kQuiet = 0x1p-32;

// v 2^(512 k)
__device__ inline double true_value(double v, int k) { return ldexp(v, kScaleStep * k); }

// One wave per (64 pairs, m).  The coefficients are uniform over the wave.
// Beside the start it finds, for the mixed forms, the first rows where a value
// passes 2^-32: below, the split-FP16 form's operands are zero.  (Padded pairs
// have no row.)
template <bool F32>
__global__ __launch_bounds__(64) void k_live_start(
    PairDesc *__restrict__ pairs, int npairs, const int *__restrict__ mval,
    const long long *__restrict__ moff, const double *__restrict__ mu, int lmax,
    const double *__restrict__ A, int np, int nb,
    double2 *__restrict__ st, uint16_t *__restrict__ je, ushort2 *__restrict__ jr,
    uint16_t *__restrict__ jq)
{
    const int blk = blockIdx.x, i = blockIdx.y;
    const int p = blk * 64 + threadIdx.x;
    const int m = mval[i], len = lmax - m + 1;
    const double *__restrict__ Am = A + moff[i];
    constexpr double t = F32 ? kFloor32 : kFloor64;
    double x = 0.0, s = 0.0;
    if (p < npairs) {
        x = pairs[p].x;
        s = pairs[p].s;
    }
    double u0, u1 = 0.0;
    int k;
    seed_mm(mu[i], s, m, u0, k);
    u0 = -u0;
    int start = kNeverLive, loud = kNeverLive;
    double2 v = make_double2(0.0, 0.0);
    for (int j = 0; j < len; j += kLiveRows) {
        const double s0 = u0, s1 = u1;
        const int sk = k;
        double big = 0.0;
#pragma unroll
        for (int q = 0; q < kLiveRows; ++q) {
            // rows past the m's end (the next m's, or the table's padding)
            // are computed and not looked at
            const double u = fma(Am[j + q] * x, u1, -u0);
            u0 = u1;
            u1 = u;
            big = (j + q < len) ? fmax(big, fabs(u)) : big;
        }
        if (start == kNeverLive && p < npairs && true_value(big, sk) > t) {
            start = j / kLiveRows;
            v = make_double2(true_value(s0, sk), true_value(s1, sk));
        }
        if (F32 && p < npairs && true_value(big, sk) > kQuiet) loud = min(loud, j / kLiveRows);
        if (fmax(fabs(u0), fabs(u1)) > kTwoS) {
            u0 *= kTwoMinusS;
            u1 *= kTwoMinusS;
            k += 1;
        }
        if (__ballot(start == kNeverLive && p < npairs) == 0 &&
            (!F32 || __ballot(loud != kNeverLive) != 0))
            break;
    }
    st[(long long)i * np + p] = v;
    je[(long long)i * np + p] = (uint16_t)start;
    int lo = start, hi = start == kNeverLive ? 0 : start;
    for (int o = 32; o >= 1; o >>= 1) {
        lo = min(lo, __shfl_xor(lo, o));
        hi = max(hi, __shfl_xor(hi, o));
        if (F32) loud = min(loud, __shfl_xor(loud, o));
    }
    if (threadIdx.x == 0) {
        jr[(long long)i * nb + blk] = make_ushort2((unsigned short)lo, (unsigned short)hi);
        if (F32) jq[(long long)i * nb + blk] = (uint16_t)loud;
    }
    if (start != kNeverLive) atomicMax(F32 ? &pairs[p].ilim32 : &pairs[p].ilim, i + 1);
}

template <bool F32>
__global__ __launch_bounds__(256) void k_live_rings(const PairDesc *__restrict__ pairs, int npairs,
                                                    const int *__restrict__ mval,
                                                    RingDesc *__restrict__ rings)
{
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= npairs) return;
    const PairDesc d = pairs[p];
    const int lim = F32 ? d.ilim32 : d.ilim;
    const int ml = lim > 0 ? mval[lim - 1] : -1;
    (F32 ? rings[d.rn].mlive32 : rings[d.rn].mlive) = ml;
    if (d.rs >= 0) (F32 ? rings[d.rs].mlive32 : rings[d.rs].mlive) = ml;
}

template <bool F32>
hipError_t live_table(const sht_plan_s *p, const LiveTab &t, hipStream_t st)
{
    hipLaunchKernelGGL(k_live_start<F32>, dim3((unsigned)t.nb, (unsigned)p->nm), dim3(64), 0, st,
                       p->d_pairs, p->npairs, p->d_mval, p->d_moff, p->d_mu, p->lmax, p->d_A,
                       t.np, t.nb, const_cast<double2 *>(t.st), const_cast<uint16_t *>(t.je),
                       const_cast<ushort2 *>(t.jr), const_cast<uint16_t *>(t.jq));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_live_rings<F32>, dim3((unsigned)((p->npairs + 255) / 256)), dim3(256), 0,
                       st, p->d_pairs, p->npairs, p->d_mval, p->d_rings);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_live_table(const sht_plan_s *p, const LiveTab &t, bool f32, hipStream_t st)
{
    return f32 ? live_table<true>(p, t, st) : live_table<false>(p, t, st);
}

}  // namespace sht
