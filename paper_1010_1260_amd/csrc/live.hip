// Start table of the Legendre recurrence (plan time).
//
// P_mm = mu_m sin^m(theta) lies far below the smallest double for most
// (m, ring): the functions of an m stay negligible up to l ~ m / sin(theta),
// then grow within a few dozen steps to order one (Sec. 2.2.2 rescales the
// recurrence through that range at run time).  Where they start to count does
// not depend on the coefficients, so the plan finds it once: for every
// (m, ring pair) the first row j = l - m, in units of kLiveRows, from which
// the values pass
//     2^-192 x the largest |P_lm| of that m over l and the plan's rings
// (and 2^-372, below which the scaled recurrence drops terms anyhow), and the
// two recurrence values there.  The transforms begin at that row, from true
// FP64 values: no rescaling, no accumulation of terms that cannot be seen,
// and nothing at all for the (m, ring) with no live row.  The dropped terms
// are smaller than an ulp of the m's sum unless coefficients of one m differ
// by more than 2^130.
//
// At l_max 4096 / nside 2048 27% of the (l, m, ring) terms are dropped
// (l_max 1024: 18%), and the table takes 18 bytes per (m, pair), 0.6 of a
// map's complex128 Delta.
#include "recurrence.h"
#include "sht_internal.h"

namespace sht {
namespace {

constexpr double kLiveFloor = 0x1p-372;
constexpr double kLiveRel = 0x1p-192;
constexpr double kQuiet = 0x1p-32;

// v 2^(512 k), 0 for k <= -2 (below 2^-372 for |v| < 2^652)
__device__ inline double true_abs(double v, int k) { return fabs(v) * final_scale(k); }

// thr[i] = max(2^-372, 2^-192 max_l |u_l|) of the pair with the largest
// sin(theta), where the functions of every m are largest at given l in the
// growing range.  One thread per m: 4097 chains of at most 4097 steps.
__global__ __launch_bounds__(64) void k_live_threshold(
    const PairDesc *__restrict__ pairs, int pmax, const int *__restrict__ mval,
    const long long *__restrict__ moff, const double *__restrict__ mu, int nm, int lmax,
    const double *__restrict__ A, double *__restrict__ thr)
{
    const int i = blockIdx.x * 64 + threadIdx.x;
    if (i >= nm) return;
    const double x = pairs[pmax].x;
    const int m = mval[i], len = lmax - m + 1;
    const double *Am = A + moff[i];
    double u0, u1 = 0.0, big;
    int k;
    seed_mm(mu[i], pairs[pmax].s, m, u0, k);
    u0 = -u0;   // u_{-2}, so that row 0 of the recurrence gives the seed
    big = true_abs(u0, k);
    for (int j = 0; j < len; ++j) {
        const double u = fma(Am[j] * x, u1, -u0);
        u0 = u1;
        u1 = u;
        big = fmax(big, true_abs(u, k));
        if ((j & 7) == 7 && fmax(fabs(u0), fabs(u1)) > kTwoS) {
            u0 *= kTwoMinusS;
            u1 *= kTwoMinusS;
            k += 1;
        }
    }
    thr[i] = fmax(kLiveFloor, kLiveRel * big);
}

// One wave per (64 pairs, m).  The coefficients are uniform over the wave.
// Beside the start it finds the first rows where a value passes 2^-32: below,
// the split-FP16 form's operands are zero.  (Padded pairs have no row.)
__global__ __launch_bounds__(64) void k_live_start(
    PairDesc *__restrict__ pairs, int npairs, const int *__restrict__ mval,
    const long long *__restrict__ moff, const double *__restrict__ mu, int lmax,
    const double *__restrict__ A, const double *__restrict__ thr, int np, int nb,
    double2 *__restrict__ st, uint16_t *__restrict__ je, ushort2 *__restrict__ jr,
    uint16_t *__restrict__ jq)
{
    const int blk = blockIdx.x, i = blockIdx.y;
    const int p = blk * 64 + threadIdx.x;
    const int m = mval[i], len = lmax - m + 1;
    const double *__restrict__ Am = A + moff[i];
    const double t = thr[i];
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
        if (start == kNeverLive && p < npairs && true_abs(big, sk) > t) {
            start = j / kLiveRows;
            const double f = final_scale(sk);
            v = make_double2(s0 * f, s1 * f);
        }
        if (p < npairs && true_abs(big, sk) > kQuiet) loud = min(loud, j / kLiveRows);
        if (fmax(fabs(u0), fabs(u1)) > kTwoS) {
            u0 *= kTwoMinusS;
            u1 *= kTwoMinusS;
            k += 1;
        }
        if (__ballot(start == kNeverLive && p < npairs) == 0 &&
            __ballot(loud != kNeverLive) != 0)
            break;
    }
    st[(long long)i * np + p] = v;
    je[(long long)i * np + p] = (uint16_t)start;
    int lo = start, hi = start == kNeverLive ? 0 : start;
    for (int o = 32; o >= 1; o >>= 1) {
        lo = min(lo, __shfl_xor(lo, o));
        hi = max(hi, __shfl_xor(hi, o));
        loud = min(loud, __shfl_xor(loud, o));
    }
    if (threadIdx.x == 0) {
        jr[(long long)i * nb + blk] = make_ushort2((unsigned short)lo, (unsigned short)hi);
        jq[(long long)i * nb + blk] = (uint16_t)loud;
    }
    if (start != kNeverLive) atomicMax(&pairs[p].ilim, i + 1);
}

__global__ __launch_bounds__(256) void k_live_rings(const PairDesc *__restrict__ pairs, int npairs,
                                                    const int *__restrict__ mval,
                                                    RingDesc *__restrict__ rings)
{
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= npairs) return;
    const PairDesc d = pairs[p];
    const int ml = d.ilim > 0 ? mval[d.ilim - 1] : -1;
    rings[d.rn].mlive = ml;
    if (d.rs >= 0) rings[d.rs].mlive = ml;
}

}  // namespace

hipError_t launch_live_table(const sht_plan_s *p, double *scratch, int pmax, hipStream_t st)
{
    const LiveTab &t = p->live;
    hipLaunchKernelGGL(k_live_threshold, dim3((unsigned)((p->nm + 63) / 64)), dim3(64), 0, st,
                       p->d_pairs, pmax, p->d_mval, p->d_moff, p->d_mu, p->nm, p->lmax, p->d_A,
                       scratch);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_live_start, dim3((unsigned)t.nb, (unsigned)p->nm), dim3(64), 0, st,
                       p->d_pairs, p->npairs, p->d_mval, p->d_moff, p->d_mu, p->lmax, p->d_A,
                       scratch, t.np, t.nb, const_cast<double2 *>(t.st),
                       const_cast<uint16_t *>(t.je), const_cast<ushort2 *>(t.jr),
                       const_cast<uint16_t *>(t.jq));
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_live_rings, dim3((unsigned)((p->npairs + 255) / 256)), dim3(256), 0, st,
                       p->d_pairs, p->npairs, p->d_mval, p->d_rings);
    return hipGetLastError();
}

}  // namespace sht
