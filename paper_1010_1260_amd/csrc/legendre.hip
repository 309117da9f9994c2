// Legendre stage of alm2map and of its adjoint, FP64, for gfx950.
//
// Forward (Eq. DeltaDef, Sec. 2.1; Algorithms 1-2 with the recurrence merged
// into the accumulation, Sec. 2.2.2):
//     Delta_m(theta_r) = sum_{l=m}^{lmax} a_lm P_lm(cos theta_r).
//
// Recurrence.  Eq. (assLegRec) with the sign that yields orthonormal
// functions, P_l = beta_l (x P_{l-1} - P_{l-2} / beta_{l-1}), is rewritten
// for u_l = P_l / c_l with c_m = c_{m+1} = 1 and c_l = (beta_l/beta_{l-1}) c_{l-2}:
//     u_l = (A_l x) u_{l-1} - u_{l-2},      A_l = beta_l c_{l-1} / c_l,
// so one step is a multiply and a fused multiply-add; c_l (between 0.17 and
// 1.13 for l <= 4096) is folded into the coefficients, a'_lm = c_lm a_lm,
// by a prescale kernel.  The seeds are P_mm = mu_m sin^m(theta) (Eq. pmm,
// exponent m/2 on 1-x^2) and P_{m+1,m} = sqrt(2m+3) x P_mm (Eq. pm1m).
//
// Start.  The values of an m are negligible up to l ~ m / sin(theta); every
// (m, ring pair) starts at the row of the plan's start table (live.hip) from
// true FP64 values, so the forward kernels neither rescale nor touch the terms
// before it.  (The adjoint still carries scaled values (v, k), value
// v 2^(512 k), k <= 0, rescaled every 16 steps, Sec. 2.2.2.)
//
// Mapping to CDNA4.  One wavefront owns 64*CH ring pairs (CH chains per
// lane) and NB maps; the north/south rings of a pair share the recurrence
// through the parity P_lm(-x) = (-1)^(l+m) P_lm(x): even l-m terms go to E,
// odd to O, Delta_N = E + O, Delta_S = E - O; the maps share it too.  (l, m)
// is uniform across the wave, so A_l and a'_lm are read with scalar loads
// into SGPRs, a chunk of rows ahead, and fed straight into the FP64 VALU ops:
// 2 + 2 NB VALU instructions per (l, m, chain) and no LDS.
// A wave processes the m-pair (m_i, m_{nm-1-i}) whose lengths sum to a
// constant, which balances the triangular work.
//
// Bound: FP64 VALU issue.  l_max 4096 / nside 2048, one map: 1.6e9 wave
// instructions, 2.6 ms at 2.4 GHz (the card runs this kernel near 2.0 GHz),
// measured 3.84 ms; 4.32 ms with the rows' loads just before their use, 5.63 ms
// with rescaled chains over all rows.  8 maps at l_max 1024 / nside 512 with
// prescale: 432 us in fours, 578 us one by one.
#include <type_traits>

#include "recurrence.h"
#include "sht_internal.h"

namespace sht {
namespace {

// a'_lm = c_lm a_lm of NB maps, interleaved [lm][map] for the waves that take
// the NB maps together.
template <int NB>
__global__ __launch_bounds__(256) void k_prescale(const double2 *__restrict__ alm,
                                                  const double *__restrict__ cn,
                                                  double2 *__restrict__ ap, long long nalm,
                                                  long long m0len)
{
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long g = (long long)blockIdx.y * NB;
    if (e >= nalm) return;
    const double c = cn[e];
    double2 a[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) a[b] = alm[(g + b) * nalm + e];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        a[b].x *= c;
        a[b].y = (e < m0len) ? 0.0 : a[b].y * c;
        ap[g * nalm + e * NB + b] = a[b];
    }
}

template <int CH>
struct Chains {
    double x[CH];
    int rn[CH], rs[CH], ilim[CH];
};

// The ring pairs of this lane's chains: 64-pair blocks blk0..blk0 + CH - 1.
template <int CH>
__device__ inline void load_chains(Chains<CH> &g, const PairDesc *__restrict__ pairs, int npairs,
                                   int blk0)
{
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int p = (blk0 + c) * 64 + (int)threadIdx.x;
        if (p < npairs) {
            const PairDesc d = pairs[p];
            g.x[c] = d.x; g.rn[c] = d.rn; g.rs[c] = d.rs; g.ilim[c] = d.ilim;
        } else {
            g.x[c] = 0.0; g.rn[c] = -1; g.rs[c] = -1; g.ilim[c] = 0;
        }
    }
}

// Wave-uniform data that no kernel writes while it reads it comes through the
// constant address space: scalar loads, also where the compiler cannot prove
// that the kernel's stores leave it alone (the batch's workspace holds both
// the coefficients and Delta).
typedef const int __attribute__((address_space(4))) *CIp;
typedef const long long __attribute__((address_space(4))) *CLp;
typedef const double __attribute__((address_space(4))) *CDp;

// The coefficients of KR rows of one m in scalar registers: A_l, and a'_lm of
// the wave's NB maps.
// (Vector-typed loads of 8-byte alignment: one s_load per 64 bytes.)
typedef double d2a __attribute__((ext_vector_type(2), aligned(8)));
typedef double d4a __attribute__((ext_vector_type(4), aligned(8)));
typedef double d8a __attribute__((ext_vector_type(8), aligned(8)));

template <int KR, int NB>
struct CoefRows {
    double A[KR], a[2 * KR * NB];   // a: [row][map][re, im]

    template <int N>
    __device__ static inline void get(double *d, CDp p)
    {
        if constexpr (N >= 8) {
            const d8a v = *(const d8a __attribute__((address_space(4))) *)p;
#pragma unroll
            for (int t = 0; t < 8; ++t) d[t] = v[t];
            if constexpr (N > 8) get<N - 8>(d + 8, p + 8);
        } else if constexpr (N >= 4) {
            const d4a v = *(const d4a __attribute__((address_space(4))) *)p;
#pragma unroll
            for (int t = 0; t < 4; ++t) d[t] = v[t];
            if constexpr (N > 4) get<N - 4>(d + 4, p + 4);
        } else {
            const d2a v = *(const d2a __attribute__((address_space(4))) *)p;
            d[0] = v[0];
            d[1] = v[1];
        }
    }
    __device__ inline void load(CDp Am, CDp am, int j)
    {
        get<KR>(A, Am + j);
        get<2 * KR * NB>(a, am + 2 * NB * j);
    }
    __device__ double re(int t, int b) const { return a[2 * (t * NB + b)]; }
    __device__ double im(int t, int b) const { return a[2 * (t * NB + b) + 1]; }
};

// One m of an m-pair for CH chains per lane and NB maps: forward accumulation.
// The recurrence of a chain is shared by the maps: 2 + 2 NB FP64 instructions
// per (l, m, pair).  ap: the maps' a'_lm, [lm][map].  full: write the Delta of
// every ring, also of the m that are dead on it (the ring stage reads the
// positions below ilim only).
//
// The rows' coefficients come in scalar loads, a chunk of KR rows ahead of
// their use: scalar loads return out of order, so a chunk is waited for as a
// whole, just before the next one is asked for.
template <int CH, int NB>
__device__ inline void fwd_one_m(const Chains<CH> &g, const LiveTab &lt, int blk0, int m, int i,
                                 long long off, int lmax, const double *__restrict__ A,
                                 const double2 *__restrict__ ap, double2 *__restrict__ delta,
                                 long long dbase, long long dmap, int nrings, bool full)
{
    constexpr int KR = NB == 1 ? 4 : 2;   // two chunks fit the scalar registers
    const int len = lmax - m + 1;
    const CDp Am = (CDp)(A + off);
    const CDp am = (CDp)(ap + off * NB);   // (re, im) pairs
    // rows [8 lo, 8 hi]: where this wave's pairs start
    int lo = kNeverLive, hi = 0;
    {
        const CIp jr = (CIp)(lt.jr + (long long)i * lt.nb);
#pragma unroll
        for (int c = 0; c < CH; ++c)
            if (blk0 + c < lt.nb) {
                const int v = jr[blk0 + c];
                lo = min(lo, v & 0xffff);
                hi = max(hi, (int)((unsigned)v >> 16));
            }
    }
    double Er[CH][NB], Ei[CH][NB], Or[CH][NB], Oi[CH][NB];
#pragma unroll
    for (int c = 0; c < CH; ++c)
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            Er[c][b] = 0.0; Ei[c][b] = 0.0; Or[c][b] = 0.0; Oi[c][b] = 0.0;
        }
    if (lo != kNeverLive) {
        double u0[CH], u1[CH], s0[CH], s1[CH];
        int je[CH];
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            u0[c] = 0.0; u1[c] = 0.0; s0[c] = 0.0; s1[c] = 0.0;
            je[c] = kNeverLive;
            if (blk0 + c < lt.nb) {
                const long long e = (long long)i * lt.np + (blk0 + c) * 64 + (int)threadIdx.x;
                const double2 v = lt.st[e];
                s0[c] = v.x; s1[c] = v.y;
                je[c] = lt.je[e];
            }
        }
        // a chain is zero until its start row, where it takes the table's values
        auto enter = [&](int jb) {
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const bool on = je[c] == jb;
                u0[c] = on ? s0[c] : u0[c];
                u1[c] = on ? s1[c] : u1[c];
            }
        };
        auto rows = [&](const CoefRows<KR, NB> &r) {
#pragma unroll
            for (int t = 0; t < KR; t += 2) {
#pragma unroll
                for (int c = 0; c < CH; ++c) {
                    const double u2 = fma(r.A[t] * g.x[c], u1[c], -u0[c]);
                    const double u3 = fma(r.A[t + 1] * g.x[c], u2, -u1[c]);
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        Er[c][b] = fma(r.re(t, b), u2, Er[c][b]);
                        Ei[c][b] = fma(r.im(t, b), u2, Ei[c][b]);
                        Or[c][b] = fma(r.re(t + 1, b), u3, Or[c][b]);
                        Oi[c][b] = fma(r.im(t + 1, b), u3, Oi[c][b]);
                    }
                    u0[c] = u2; u1[c] = u3;
                }
            }
        };
        int j = lo * kLiveRows;
        const int jhi = hi * kLiveRows;
        if (j + 8 <= len) {
            CoefRows<KR, NB> ca, cb;
            ca.load(Am, am, j);
            // s_waitcnt lgkmcnt(0), and nothing moves across
            auto arrived = [] {
                __builtin_amdgcn_sched_barrier(0);
                __builtin_amdgcn_s_waitcnt(0xC07F);
                __builtin_amdgcn_sched_barrier(0);
            };
            auto rows8 = [&](int jn) {   // rows j..j + 7; jn: the rows wanted next
#pragma unroll
                for (int t = 0; t < 8; t += 2 * KR) {
                    arrived();
                    cb.load(Am, am, j + t + KR);
                    __builtin_amdgcn_sched_barrier(0);
                    rows(ca);
                    arrived();
                    ca.load(Am, am, t + 2 * KR < 8 ? j + t + 2 * KR : jn);
                    __builtin_amdgcn_sched_barrier(0);
                    rows(cb);
                }
            };
            // the last chunk's look-ahead stays inside the m
            for (; j <= jhi && j + 8 <= len; j += 8) {
                enter(j / kLiveRows);
                rows8(min(j + 8, len - KR));
            }
            for (; j + 8 <= len; j += 8) rows8(min(j + 8, len - KR));
        }
        if (j < len) {
            enter(j / kLiveRows);
            for (; j < len; ++j) {
                const double Aa = Am[j];
                const bool odd = j & 1;
#pragma unroll
                for (int c = 0; c < CH; ++c) {
                    const double u2 = fma(Aa * g.x[c], u1[c], -u0[c]);
                    u0[c] = u1[c]; u1[c] = u2;
                }
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    const double ar = am[2 * (j * NB + b)], ai = am[2 * (j * NB + b) + 1];
#pragma unroll
                    for (int c = 0; c < CH; ++c) {
                        if (odd) {
                            Or[c][b] = fma(ar, u1[c], Or[c][b]);
                            Oi[c][b] = fma(ai, u1[c], Oi[c][b]);
                        } else {
                            Er[c][b] = fma(ar, u1[c], Er[c][b]);
                            Ei[c][b] = fma(ai, u1[c], Ei[c][b]);
                        }
                    }
                }
            }
        }
    }
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        if (!full && i >= g.ilim[c]) continue;
        double2 *row = delta + dbase + (long long)i * nrings;
#pragma unroll
        for (int b = 0; b < NB; ++b, row += dmap) {
            // Delta [m][ring]: consecutive lanes write consecutive rings
            if (g.rn[c] >= 0)
                row[g.rn[c]] = make_double2(Er[c][b] + Or[c][b], Ei[c][b] + Oi[c][b]);
            if (g.rs[c] >= 0)
                row[g.rs[c]] = make_double2(Er[c][b] - Or[c][b], Ei[c][b] - Oi[c][b]);
        }
    }
}

// groups of NB maps from the first map of ap and delta on
template <int CH, int NB>
__global__ __launch_bounds__(64) void k_legendre_fwd(
    const PairDesc *__restrict__ pairs, int npairs, LiveTab lt, int pblocks,
    const int *__restrict__ mval, const long long *__restrict__ moff, int nm, int nmpairs,
    int lmax, const double *__restrict__ A, const double2 *__restrict__ ap, long long nalm,
    double2 *__restrict__ delta, int nrings, int ngroups, int full)
{
    // XCD x takes the m-pairs q = x mod 8, one after the other for all ring
    // blocks of all maps: the waves that share an m-pair's coefficients run
    // together on one L2, and since the live rows of an m-pair shrink with q
    // (by half from q = 0 to the last), every XCD gets the same share of them.
    const int x = (int)(blockIdx.x % 8);
    const int w = (int)(blockIdx.x / 8);
    const int pb = w % pblocks;
    const int rest = w / pblocks;
    const long long b = (long long)(rest % ngroups) * NB;
    const int q = x + 8 * (rest / ngroups);
    if (q >= nmpairs) return;

    Chains<CH> g;
    load_chains(g, pairs, npairs, pb * CH);
    const double2 *apb = ap + b * nalm;
    const long long dmap = (long long)nrings * nm;
    for (int t = 0; t < 2; ++t) {
        const int i = (t == 0) ? q : nm - 1 - q;
        if (t == 1 && i == q) break;
        fwd_one_m<CH, NB>(g, lt, pb * CH, ((CIp)mval)[i], i, ((CLp)moff)[i], lmax, A, apb, delta,
                          b * dmap, dmap, nrings, full != 0);
    }
}

// ------------------------------------------------------------------ adjoint
//
// out_lm = c_lm sum_pairs u_l(x_p) (Dt_N + (-1)^(l-m) Dt_S) 2^(512 k_l)
// A wave owns 64*CH ring pairs and one m-pair; per tile of 16 l-values each
// lane sums its chains, the 64 lane partials go through LDS (16 x 64
// complex, wave-private) and are reduced to one partial per (ring block, l).
// A second kernel adds the ring-block partials in a fixed order and applies
// c_lm, so the result is bitwise reproducible.

constexpr int kAdjTile = 16;
// Row length of the reduction buffer: 64 lane partials plus one pad entry.
// The reduction reads a column (lanes 0..15 take rows 0..15); with rows of
// exactly 64 entries (1 KB) those reads would all fall in one LDS bank.
constexpr int kAdjRow = 65;

template <int CH>
__device__ inline void adj_one_m(const Chains<CH> &g, const double (&s)[CH], int m, int i,
                                 long long off, double mum, int lmax,
                                 const double *__restrict__ A,
                                 const double2 *__restrict__ dt, long long dtbase, int nrings,
                                 double2 *__restrict__ part, double2 (*red)[kAdjRow])
{
    const int len = lmax - m + 1;
    const int lane = threadIdx.x;
    const double *__restrict__ Am = A + off;
    double u0[CH], u1[CH];
    double WEr[CH], WEi[CH], WOr[CH], WOi[CH];  // pair weights times 2^(512 k) factor
    double NEr[CH], NEi[CH], NOr[CH], NOi[CH];  // unscaled pair weights
    int k[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        double2 wn = make_double2(0.0, 0.0), ws = make_double2(0.0, 0.0);
        if (g.rn[c] >= 0) wn = dt[dtbase + (long long)i * nrings + g.rn[c]];
        if (g.rs[c] >= 0) ws = dt[dtbase + (long long)i * nrings + g.rs[c]];
        NEr[c] = wn.x + ws.x; NEi[c] = wn.y + ws.y;
        NOr[c] = wn.x - ws.x; NOi[c] = wn.y - ws.y;
        seed_mm(mum, s[c], m, u0[c], k[c]);
        u1[c] = (len >= 2) ? (Am[1] * g.x[c]) * u0[c] : 0.0;
        const double f = final_scale(k[c]);
        WEr[c] = NEr[c] * f; WEi[c] = NEi[c] * f; WOr[c] = NOr[c] * f; WOi[c] = NOi[c] * f;
    }
    for (int j0 = 0; j0 < len; j0 += kAdjTile) {
        double pr[kAdjTile], pi[kAdjTile];
#pragma unroll
        for (int t = 0; t < kAdjTile; ++t) { pr[t] = 0.0; pi[t] = 0.0; }
#pragma unroll
        for (int t = 0; t < kAdjTile; ++t) {
            const int j = j0 + t;
            if (j < len) {
                const double Aj = (j >= 2) ? Am[j] : 0.0;
#pragma unroll
                for (int c = 0; c < CH; ++c) {
                    double u;
                    if (j == 0) {
                        u = u0[c];
                    } else if (j == 1) {
                        u = u1[c];
                    } else {
                        u = fma(Aj * g.x[c], u1[c], -u0[c]);
                        u0[c] = u1[c]; u1[c] = u;
                    }
                    if (t & 1) {  // j0 is even, so t carries the parity of l - m
                        pr[t] = fma(u, WOr[c], pr[t]);
                        pi[t] = fma(u, WOi[c], pi[t]);
                    } else {
                        pr[t] = fma(u, WEr[c], pr[t]);
                        pi[t] = fma(u, WEi[c], pi[t]);
                    }
                }
            }
        }
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            if (fmax(fabs(u0[c]), fabs(u1[c])) > kTwoS) {
                u0[c] *= kTwoMinusS; u1[c] *= kTwoMinusS;
                k[c] += 1;
                const double f = final_scale(k[c]);
                WEr[c] = NEr[c] * f; WEi[c] = NEi[c] * f;
                WOr[c] = NOr[c] * f; WOi[c] = NOi[c] * f;
            }
        }
#pragma unroll
        for (int t = 0; t < kAdjTile; ++t) red[t][lane] = make_double2(pr[t], pi[t]);
        __syncthreads();
        {
            const int t = lane & (kAdjTile - 1);
            const int seg = lane / kAdjTile;  // 4 segments of 16 lanes
            double sr = 0.0, si = 0.0;
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                const double2 v = red[t][seg * 16 + q];
                sr += v.x; si += v.y;
            }
            sr += __shfl_xor(sr, 16); si += __shfl_xor(si, 16);
            sr += __shfl_xor(sr, 32); si += __shfl_xor(si, 32);
            if (seg == 0 && j0 + t < len) part[off + j0 + t] = make_double2(sr, si);
        }
        __syncthreads();
    }
}

template <int CH>
__global__ __launch_bounds__(64) void k_legendre_adj(
    const PairDesc *__restrict__ pairs, int npairs, int pblocks,
    const int *__restrict__ mval, const long long *__restrict__ moff,
    const double *__restrict__ mu, int nm, int nmpairs, int lmax,
    const double *__restrict__ A, const double2 *__restrict__ dt, int nrings,
    double2 *__restrict__ part, long long nalm, long long total)
{
    __shared__ double2 red[kAdjTile][kAdjRow];
    const long long L = xcd_logical(blockIdx.x, total);
    const int pb = (int)(L % pblocks);
    const long long rest = L / pblocks;
    const int q = (int)(rest % nmpairs);
    const int b = (int)(rest / nmpairs);
    const int lane = threadIdx.x;
    Chains<CH> g;
    double s[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int p = (pb * CH + c) * 64 + lane;
        if (p < npairs) {
            const PairDesc d = pairs[p];
            g.x[c] = d.x; s[c] = d.s; g.rn[c] = d.rn; g.rs[c] = d.rs; g.ilim[c] = d.ilim;
        } else {
            g.x[c] = 0.0; s[c] = 0.0; g.rn[c] = -1; g.rs[c] = -1; g.ilim[c] = 0;
        }
    }
    const long long dtbase = (long long)b * nrings * nm;
    double2 *pp = part + ((long long)b * pblocks + pb) * nalm;
    for (int t = 0; t < 2; ++t) {
        const int i = (t == 0) ? q : nm - 1 - q;
        if (t == 1 && i == q) break;
        adj_one_m<CH>(g, s, mval[i], i, moff[i], mu[i], lmax, A, dt, dtbase, nrings, pp, red);
    }
}

__global__ void k_adj_reduce(const double2 *__restrict__ part, const double *__restrict__ cn,
                             double *__restrict__ alm, long long nalm, int pblocks,
                             long long m0len, int accumulate)
{
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long b = blockIdx.y;
    if (e >= nalm) return;
    double sr = 0.0, si = 0.0;
    const double2 *p = part + b * pblocks * nalm + e;
    for (int k = 0; k < pblocks; ++k) {
        const double2 v = p[(long long)k * nalm];
        sr += v.x; si += v.y;
    }
    const double c = cn[e];
    double2 *o = reinterpret_cast<double2 *>(alm) + b * nalm + e;
    const double2 v = make_double2(sr * c, (e < m0len) ? 0.0 : si * c);
    if (accumulate) {
        const double2 a = *o;
        *o = make_double2(a.x + v.x, a.y + v.y);
    } else {
        *o = v;
    }
}

// ---------------------------------------------------------------- batches
//
// A batch of single-map FP64 plans of different l_max / geometry runs the
// Legendre stage in one persistent launch: a fixed grid of waves takes
// tiles (map, m-pair, ring-pair block) from a work list sorted longest
// first, through an atomic counter.  The counter only hands out work; every
// tile's arithmetic is the same as in the single-plan kernel, so results do
// not depend on the schedule.  The counter is reset by a one-thread kernel
// launched before the persistent kernel (no memset node, so the sequence can
// be captured into a graph).

__global__ void k_batch_reset(int *counter) { *counter = 0; }

__global__ void k_batch_prescale(const BatchMap *__restrict__ maps,
                                 const double *const *__restrict__ alms, char *__restrict__ ws)
{
    const BatchMap &bm = maps[blockIdx.y];
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= bm.nalm) return;
    const double2 *a = reinterpret_cast<const double2 *>(alms[blockIdx.y]);
    double2 v = a[e];
    const double c = bm.cn[e];
    v.x *= c;
    v.y = (e < bm.m0len) ? 0.0 : v.y * c;
    reinterpret_cast<double2 *>(ws + bm.ap_off)[e] = v;
}

template <int CH>
__global__ __launch_bounds__(64) void k_legendre_fwd_batch(const BatchTile *__restrict__ tiles,
                                                           int ntiles,
                                                           const BatchMap *__restrict__ maps,
                                                           char *__restrict__ ws,
                                                           int *__restrict__ counter)
{
    const int lane = threadIdx.x;
    for (;;) {
        int t = 0;
        if (lane == 0) t = atomicAdd(counter, 1);
        // wave-uniform tile index: the tile, its plan's tables and every
        // coefficient of the recurrence then come through scalar loads, as
        // in the single-plan kernel
        t = __builtin_amdgcn_readfirstlane(__shfl(t, 0));
        if (t >= ntiles) break;
        const BatchTile tile = tiles[t];
        const BatchMap &bm = maps[tile.map];
        Chains<CH> g;
        load_chains(g, bm.pairs, bm.npairs, tile.pblock * CH);
        const double2 *ap = reinterpret_cast<const double2 *>(ws + bm.ap_off);
        double2 *delta = reinterpret_cast<double2 *>(ws + bm.delta_off);
        const int q = tile.mpair;
        for (int u = 0; u < 2; ++u) {
            const int i = (u == 0) ? q : bm.nm - 1 - q;
            if (u == 1 && i == q) break;
            fwd_one_m<CH, 1>(g, bm.live, tile.pblock * CH, ((CIp)bm.mval)[i], i,
                             ((CLp)bm.moff)[i], bm.lmax, bm.A, ap, delta, 0, 0, bm.nrings, false);
        }
    }
}

// The adjoint reduces every 16 l-rows over the wave's lanes through LDS.
// Four ring pairs per lane keep that reduction small next to the recurrence
// and leave registers for two waves per SIMD (224 VGPRs); at l_max 4096 the
// map2alm built on it takes 11.9 ms, against 13.8 ms with eight pairs (one
// wave per SIMD) and 16.7 ms with two.
constexpr int kAdjChains = 4;

}  // namespace

// Calls f(first map, groups, std::integral_constant of the group size) for
// the plan's maps in groups of p->fwd_group, and for the maps left over.
template <typename F>
static hipError_t for_map_groups(const sht_plan_s *p, const F &f)
{
    auto one = [&](int first, int groups, int nb) {
        switch (nb) {
        case 1: return f(first, groups, std::integral_constant<int, 1>());
        case 2: return f(first, groups, std::integral_constant<int, 2>());
        case 3: return f(first, groups, std::integral_constant<int, 3>());
        case 4: return f(first, groups, std::integral_constant<int, 4>());
        default: return hipErrorInvalidValue;
        }
    };
    const int nb = p->fwd_group, groups = p->nmaps / nb, rest = p->nmaps - groups * nb;
    hipError_t e = one(0, groups, nb);
    if (e == hipSuccess && rest > 0) e = one(groups * nb, 1, rest);
    return e;
}

hipError_t launch_prescale(const sht_plan_s *p, const double *alm, double2 *ap, hipStream_t st)
{
    const long long m0len = (p->mval[0] == 0) ? (p->lmax + 1) : 0;
    return for_map_groups(p, [&](int first, int groups, auto nb) {
        dim3 grid((unsigned)((p->nalm + 255) / 256), (unsigned)groups);
        hipLaunchKernelGGL(k_prescale<decltype(nb)::value>, grid, dim3(256), 0, st,
                           reinterpret_cast<const double2 *>(alm) + first * p->nalm, p->d_cn,
                           ap + first * p->nalm, p->nalm, m0len);
        return hipGetLastError();
    });
}

int fwd_pblocks(const sht_plan_s *p)
{
    const int per = 64 * p->fwd_chains;
    return (p->npairs + per - 1) / per;
}
int adj_pblocks(const sht_plan_s *p) { return (p->npairs + 64 * kAdjChains - 1) / (64 * kAdjChains); }

template <int NB>
static auto fwd_kernel(int chains) -> decltype(&k_legendre_fwd<1, NB>)
{
    return chains == 1   ? k_legendre_fwd<1, NB>
           : chains == 2 ? k_legendre_fwd<2, NB>
           : chains == 4 ? k_legendre_fwd<4, NB>
                         : nullptr;
}

hipError_t launch_legendre_fwd(const sht_plan_s *p, const double2 *ap, double2 *delta, bool full,
                               hipStream_t st)
{
    const int pblocks = fwd_pblocks(p);
    const int nmpairs = (p->nm + 1) / 2;
    return for_map_groups(p, [&](int first, int groups, auto nb) {
        const long long total = 8LL * ((nmpairs + 7) / 8) * pblocks * groups;
        if (total <= 0 || total > 0x7fffffffLL) return hipErrorInvalidConfiguration;
        const auto kern = fwd_kernel<decltype(nb)::value>(p->fwd_chains);
        if (!kern) return hipErrorInvalidValue;
        hipLaunchKernelGGL(kern, dim3((unsigned)total), dim3(64), 0, st, p->d_pairs, p->npairs,
                           p->live, pblocks, p->d_mval, p->d_moff, p->nm, nmpairs, p->lmax, p->d_A,
                           ap + first * p->nalm, p->nalm,
                           delta + (long long)first * p->nrings * p->nm, p->nrings, groups,
                           full ? 1 : 0);
        return hipGetLastError();
    });
}

size_t adj_part_bytes(const sht_plan_s *p)
{
    return (size_t)p->nmaps * (size_t)adj_pblocks(p) * (size_t)p->nalm * sizeof(double2);
}

hipError_t launch_legendre_adj_ws(const sht_plan_s *p, const double2 *dt, double2 *part,
                                  double *alm, hipStream_t st, bool accumulate)
{
    const int pblocks = adj_pblocks(p);
    const int nmpairs = (p->nm + 1) / 2;
    const long long total = (long long)pblocks * nmpairs * p->nmaps;
    if (total <= 0 || total > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(k_legendre_adj<kAdjChains>, dim3((unsigned)total), dim3(64), 0, st,
                       p->d_pairs, p->npairs, pblocks, p->d_mval, p->d_moff, p->d_mu, p->nm,
                       nmpairs, p->lmax, p->d_A, dt, p->nrings, part, p->nalm, total);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const long long m0len = (p->mval[0] == 0) ? (p->lmax + 1) : 0;
    dim3 grid((unsigned)((p->nalm + 255) / 256), (unsigned)p->nmaps);
    hipLaunchKernelGGL(k_adj_reduce, grid, dim3(256), 0, st, part, p->d_cn, alm, p->nalm,
                       pblocks, m0len, accumulate ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_batch_legendre(const BatchMap *maps, int nmaps, long long max_nalm,
                                 const BatchTile *tiles, int ntiles, int chains, int grid_waves,
                                 const double *const *alms, void *ws, int *counter,
                                 hipStream_t st)
{
    dim3 pg((unsigned)((max_nalm + 255) / 256), (unsigned)nmaps);
    hipLaunchKernelGGL(k_batch_prescale, pg, dim3(256), 0, st, maps, alms, (char *)ws);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_batch_reset, dim3(1), dim3(1), 0, st, counter);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    switch (chains) {
    case 1:
        hipLaunchKernelGGL(k_legendre_fwd_batch<1>, dim3((unsigned)grid_waves), dim3(64), 0, st,
                           tiles, ntiles, maps, (char *)ws, counter);
        break;
    case 2:
        hipLaunchKernelGGL(k_legendre_fwd_batch<2>, dim3((unsigned)grid_waves), dim3(64), 0, st,
                           tiles, ntiles, maps, (char *)ws, counter);
        break;
    case 4:
        hipLaunchKernelGGL(k_legendre_fwd_batch<4>, dim3((unsigned)grid_waves), dim3(64), 0, st,
                           tiles, ntiles, maps, (char *)ws, counter);
        break;
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace sht
