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
// true FP64 values, so the kernels neither rescale nor touch the terms before
// it.
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
// Bound: FP64 VALU issue.  l_max 4096 / nside 2048, one map: 1.8e9 wave
// instructions, 2.9 ms at 2.4 GHz (the card runs this kernel near 2.0 GHz),
// measured 3.97 ms; 5.63 ms with rescaled chains over all rows.  (With a start
// table that leaves out what is below 2^-192 of an m's largest value 3.61 ms,
// 4.32 with the rows' loads just before their use; but live.hip.)  8 maps at
// l_max 1024 / nside 512: 475 us in fours.
#include <type_traits>

#include "recurrence.h"
#include "sht_internal.h"

namespace sht {
namespace {

// Infinite and NaN inputs.  A coefficient that is one makes its map so on every
// ring, and a pixel every coefficient, as a sum over all terms does; the start
// table leaves terms out.  So the prescale notes which blocks of coefficients
// hold one, and the wave that has the set's first m, which no ring leaves out
// (PairDesc::ilim), adds it to that m's Delta.  The adjoint's first m of a ring
// is NaN with any pixel of it: the wave that has that m notes it for its ring
// block, and the block sum adds it to every coefficient.

__host__ __device__ inline long long bad_stride(int nbad) { return (nbad + 15LL) / 16 * 16; }

// The wave's NB flags to a workgroup's one byte.
template <int NB>
__device__ inline void store_bad(unsigned f, unsigned char *__restrict__ to)
{
    __shared__ unsigned any;
    if (threadIdx.x == 0) any = 0;
    __syncthreads();
    unsigned w = 0;
#pragma unroll
    for (int b = 0; b < NB; ++b) w |= __ballot(f >> b & 1u) ? 1u << b : 0u;
    if (w && (threadIdx.x & 63) == 0) atomicOr(&any, w);
    __syncthreads();
    if (threadIdx.x == 0) *to = (unsigned char)any;
}

// a'_lm = c_lm a_lm of NB maps, interleaved [lm][map] for the waves that take
// the NB maps together.  bad[k] (if given; the groups of maps bad_stride(nbad)
// apart): bit b is set if any of block k's 256 a'_lm of map b is infinite or NaN.
template <int NB>
__global__ __launch_bounds__(256) void k_prescale(const double2 *__restrict__ alm,
                                                  const double *__restrict__ cn,
                                                  double2 *__restrict__ ap, long long nalm,
                                                  long long m0len, int nbad,
                                                  unsigned char *__restrict__ bad)
{
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long g = (long long)blockIdx.y * NB;
    unsigned f = 0;
    if (e < nalm) {
        const double c = cn[e];
        double2 a[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) a[b] = alm[(g + b) * nalm + e];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            a[b].x *= c;
            a[b].y = (e < m0len) ? 0.0 : a[b].y * c;
            ap[g * nalm + e * NB + b] = a[b];
            f |= (isfinite(a[b].x) && isfinite(a[b].y)) ? 0u : 1u << b;
        }
    }
    if (!bad) return;
    store_bad<NB>(f, bad + blockIdx.y * bad_stride(nbad) + blockIdx.x);
}

template <int CH>
struct Chains {
    double x[CH];
    int rn[CH], rs[CH], ilim[CH];
};

// The ring pairs of this lane's chains: 64-pair blocks blk0..blk0 + CH - 1
// (the pairs are padded like the start table).
template <int CH>
__device__ inline void load_chains(Chains<CH> &g, const PairDesc *__restrict__ pairs, int blk0)
{
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const PairDesc d = pairs[(blk0 + c) * 64 + (int)threadIdx.x];
        g.x[c] = d.x; g.rn[c] = d.rn; g.rs[c] = d.rs; g.ilim[c] = d.ilim;
    }
}

// The coefficients of KR rows of one m in scalar registers: A_l, and a'_lm of
// the wave's NB maps.
template <int KR, int NB>
struct CoefRows {
    double A[KR], a[2 * KR * NB];   // a: [row][map][re, im]

    __device__ inline void load(CDp Am, CDp am, int j)
    {
        scalar_rows<KR>(A, Am + j);
        scalar_rows<2 * KR * NB>(a, am + 2 * NB * j);
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
                                 const DeltaLayout &dl, bool full, int nbad,
                                 const unsigned char *__restrict__ bad)
{
    constexpr int KR = NB == 1 ? 4 : 2;   // two chunks fit the scalar registers
    const int lane = (int)threadIdx.x;
    const int len = lmax - m + 1;
    const CDp Am = (CDp)(A + off);
    const CDp am = (CDp)(ap + off * NB);   // (re, im) pairs
    // rows [8 lo, 8 hi]: where this wave's pairs start
    int lo = kNeverLive, hi = 0;
    {
        const CIp jr = (CIp)(lt.jr + (long long)i * lt.nb);
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int v = jr[blk0 + c];
            lo = min(lo, v & 0xffff);
            hi = max(hi, (int)((unsigned)v >> 16));
        }
    }
    // the maps with an infinite or NaN coefficient: any, with the set's first m;
    // or, where every m is written, those in the rows of this m that are not
    // read below
    unsigned f = 0;
    if (full) {
        for (int j = lane; j < min(lo * kLiveRows, len); j += 64)
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const double2 v = ap[(off + j) * NB + b];
                f |= (isfinite(v.x) && isfinite(v.y)) ? 0u : 1u << b;
            }
    } else if (i == 0) {
        // 16 flags a load: the walk is on the critical path of a few waves
        const uint4 *b16 = reinterpret_cast<const uint4 *>(bad);
        for (int k = lane; k < nbad / 16; k += 64) {
            const uint4 v = b16[k];
            f |= v.x | v.y | v.z | v.w;
        }
        if (lane < nbad % 16) f |= bad[nbad - 1 - lane];
        f |= f >> 16;
        f |= f >> 8;
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
            u0[c] = 0.0; u1[c] = 0.0;
            const long long e = (long long)i * lt.np + (blk0 + c) * 64 + (int)threadIdx.x;
            const double2 v = lt.st[e];
            s0[c] = v.x; s1[c] = v.y;
            je[c] = lt.je[e];
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
            auto rows8 = [&](int jn) {   // rows j..j + 7; jn: the rows wanted next
#pragma unroll
                for (int t = 0; t < 8; t += 2 * KR) {
                    scalars_arrived();
                    cb.load(Am, am, j + t + KR);
                    __builtin_amdgcn_sched_barrier(0);
                    rows(ca);
                    scalars_arrived();
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
    if (full || i == 0) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
            if (__ballot(f >> b & 1u)) {
#pragma unroll
                for (int c = 0; c < CH; ++c) Er[c][b] = Ei[c][b] = __builtin_nan("");
            }
    }
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        if (!full && i >= g.ilim[c]) continue;
        // consecutive lanes write consecutive rings
        double2 *n = delta + dl.row(max(g.rn[c], 0)) + i * dl.mstride(g.rn[c]);
        double2 *so = delta + dl.row(max(g.rs[c], 0)) + i * dl.mstride(g.rs[c]);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            if (g.rn[c] >= 0)
                n[b * dl.map] = make_double2(Er[c][b] + Or[c][b], Ei[c][b] + Oi[c][b]);
            if (g.rs[c] >= 0)
                so[b * dl.map] = make_double2(Er[c][b] - Or[c][b], Ei[c][b] - Oi[c][b]);
        }
    }
}

// groups of NB maps from the first map of ap and delta on
template <int CH, int NB>
__global__ __launch_bounds__(64) void k_legendre_fwd(
    const PairDesc *__restrict__ pairs, LiveTab lt, int pblocks,
    const int *__restrict__ mval, const long long *__restrict__ moff, int nm, int nmpairs,
    int lmax, const double *__restrict__ A, const double2 *__restrict__ ap, long long nalm,
    double2 *__restrict__ delta, DeltaLayout dl, int ngroups, int full, int nbad,
    const unsigned char *__restrict__ bad)
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
    load_chains(g, pairs, pb * CH);
    const double2 *apb = ap + b * nalm;
    for (int t = 0; t < 2; ++t) {
        const int i = (t == 0) ? q : nm - 1 - q;
        if (t == 1 && i == q) break;
        fwd_one_m<CH, NB>(g, lt, pb * CH, ((CIp)mval)[i], i, ((CLp)moff)[i], lmax, A, apb,
                          delta + b * dl.map, dl, full != 0, nbad,
                          bad + (rest % ngroups) * bad_stride(nbad));
    }
}

// ------------------------------------------------------------------ adjoint
//
// out_lm = c_lm sum_pairs u_l(x_p) (Dt_N + (-1)^(l-m) Dt_S).
// A wave owns 64*CH ring pairs and one m-pair and walks the rows l - m in
// tiles of 16, each chain from its start row (live.hip) on.  Chain after
// chain adds its tile to the lane's 32 partial sums (16 rows, re and im): two
// instructions of recurrence and two of accumulation per row, A_l from scalar
// registers (the next tile's asked for a tile ahead).  The 32 sums are then
// reduced over the 64 lanes in registers, halving the values and the lanes
// that hold one at each step (reduce_tile), and one partial per (ring block,
// l) is written; a second kernel adds the ring blocks' partials in a fixed
// order and applies c_lm, so the result is bitwise reproducible.
//
// The reduction costs 124 instructions per tile whatever CH, against 64 per
// chain: more chains per lane make it cheap, but leave fewer waves.
//
// Bound: VALU issue.  l_max 4096 / nside 2048, one map, with the block sum: 6.47
// ms (10.47 ms with the lanes' partials reduced through LDS, four chains and
// every row from l = m on); l_max 1024 / nside 512, 8 maps: 927 us (1405).
constexpr int kAdjTile = 16;

__device__ inline double2 halves_swapped(double a, double b, bool rows16)
{
    const unsigned al = __double2loint(a), ah = __double2hiint(a);
    const unsigned bl = __double2loint(b), bh = __double2hiint(b);
    typedef unsigned v2u __attribute__((ext_vector_type(2)));
    const v2u l = rows16 ? __builtin_amdgcn_permlane16_swap(al, bl, false, false)
                         : __builtin_amdgcn_permlane32_swap(al, bl, false, false);
    const v2u h = rows16 ? __builtin_amdgcn_permlane16_swap(ah, bh, false, false)
                         : __builtin_amdgcn_permlane32_swap(ah, bh, false, false);
    return make_double2(__hiloint2double((int)h[0], (int)l[0]),
                        __hiloint2double((int)h[1], (int)l[1]));
}

template <int CTRL>
__device__ inline double dpp(double v)
{
    const int l = __double2loint(v), h = __double2hiint(v);
    return __hiloint2double(__builtin_amdgcn_update_dpp(h, h, CTRL, 0xf, 0xf, false),
                            __builtin_amdgcn_update_dpp(l, l, CTRL, 0xf, 0xf, false));
}

// Lanes with `up` go on with b, the others with a; each adds the value of its
// partner lane, whose `up` is the opposite.
template <int CTRL>
__device__ inline double take_half(double a, double b, bool up)
{
    const double keep = up ? b : a, send = up ? a : b;
    return keep + dpp<CTRL>(send);
}

// v[k] of all lanes -> lane 2 k (and 2 k + 1) holds the sum of v[k] over the
// wave, in a fixed order.
__device__ inline double reduce_tile(double (&v)[2 * kAdjTile], int lane)
{
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const double2 t = halves_swapped(v[k], v[k + 16], false);
        v[k] = t.x + t.y;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const double2 t = halves_swapped(v[k], v[k + 8], true);
        v[k] = t.x + t.y;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = take_half<0x128>(v[k], v[k + 4], lane & 8);   // row_ror:8
#pragma unroll
    for (int k = 0; k < 2; ++k) v[k] = take_half<0x141>(v[k], v[k + 2], lane & 4);   // half mirror
    v[0] = take_half<0x4e>(v[0], v[1], lane & 2);                                    // quad xor 2
    return v[0] + dpp<0xb1>(v[0]);                                                   // quad xor 1
}

// First row of the tiles that a wave of CH 64-pair blocks writes for an m, from
// the blocks' start rows; past any row if none is live.
template <int CH>
__device__ inline int adj_first_row(CIp jr, int blk0)
{
    int lo = kNeverLive;
#pragma unroll
    for (int c = 0; c < CH; ++c) lo = min(lo, jr[blk0 + c] & 0xffff);
    return (lo * kLiveRows) & ~(kAdjTile - 1);
}

template <int CH>
__device__ inline void adj_one_m(const PairDesc *__restrict__ pairs, const LiveTab &lt,
                                 int blk0, int m, int i, long long off,
                                 int lmax, const double *__restrict__ A,
                                 const double2 *__restrict__ dt, const DeltaLayout &dl,
                                 double2 *__restrict__ part, double2 (*st)[64],
                                 int *__restrict__ bad)
{
    const int len = lmax - m + 1;
    const int lane = threadIdx.x;
    const CIp jr = (CIp)(lt.jr + (long long)i * lt.nb);
    const CDp Am = (CDp)(A + off);
    int j0 = adj_first_row<CH>(jr, blk0);
    if (j0 >= len && !bad) return;
    int lo[CH], hi[CH];    // rows where the block's pairs start
    int je[CH];
    double x[CH], u0[CH], u1[CH];
    double WEr[CH], WEi[CH], WOr[CH], WOi[CH];
    // all loads of the chains first, the pairs' before the Delta~ that they
    // place: entries that are dead or have no mirror ring are read from a
    // place in the table and dropped
    PairDesc d[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) d[c] = pairs[(blk0 + c) * 64 + lane];
    double2 sv[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int v = jr[blk0 + c];
        lo[c] = (v & 0xffff) * kLiveRows;
        hi[c] = (int)((unsigned)v >> 16) * kLiveRows;
        const long long e = (long long)i * lt.np + (blk0 + c) * 64 + lane;
        je[c] = lt.je[e];
        sv[c] = lt.st[e];
    }
    double2 wn[CH], ws[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int rn = max(d[c].rn, 0), rs = d[c].rs >= 0 ? d[c].rs : rn;
        wn[c] = dt[dl.row(rn) + i * dl.mstride(rn)];
        ws[c] = dt[dl.row(rs) + i * dl.mstride(rs)];
    }
    if (bad) {   // the dead ones too
        bool f = false;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const bool fin = isfinite(wn[c].x) && isfinite(wn[c].y) && isfinite(ws[c].x) &&
                             isfinite(ws[c].y);
            f = f || (d[c].rn >= 0 && !fin);
        }
        const int any = __ballot(f) != 0;
        if (lane == 0) *bad = any;
        if (j0 >= len) return;
    }
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        st[c][lane] = sv[c];
        x[c] = d[c].x;
        u0[c] = 0.0;
        u1[c] = 0.0;
        const bool live = i < d[c].ilim, two = live && d[c].rs >= 0;
        const double nr = live ? wn[c].x : 0.0, ni = live ? wn[c].y : 0.0;
        const double sr = two ? ws[c].x : 0.0, si = two ? ws[c].y : 0.0;
        WEr[c] = nr + sr; WEi[c] = ni + si;
        WOr[c] = nr - sr; WOi[c] = ni - si;
    }
    // a chain is zero until its start row
    auto enter = [&](int c, int jb) {
        if (je[c] == jb) {
            const double2 v = st[c][lane];
            u0[c] = v.x;
            u1[c] = v.y;
        }
    };
    double a[kAdjTile];
    scalar_rows<kAdjTile>(a, Am + j0);
    for (; j0 < len; j0 += kAdjTile) {
        // rows past the m's end (the table is padded) are computed and not stored
        double an[kAdjTile], v[2 * kAdjTile];
        scalars_arrived();
        scalar_rows<kAdjTile>(an, Am + j0 + kAdjTile);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < 2 * kAdjTile; ++t) v[t] = 0.0;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            if (lo[c] >= j0 + kAdjTile) continue;
#pragma unroll
            for (int h = 0; h < kAdjTile; h += kLiveRows) {
                if (j0 + h <= hi[c]) enter(c, (j0 + h) / kLiveRows);
#pragma unroll
                for (int t = h; t < h + kLiveRows; t += 2) {
                    u0[c] = fma(a[t] * x[c], u1[c], -u0[c]);
                    v[2 * t] = fma(u0[c], WEr[c], v[2 * t]);
                    v[2 * t + 1] = fma(u0[c], WEi[c], v[2 * t + 1]);
                    u1[c] = fma(a[t + 1] * x[c], u0[c], -u1[c]);
                    v[2 * t + 2] = fma(u1[c], WOr[c], v[2 * t + 2]);
                    v[2 * t + 3] = fma(u1[c], WOi[c], v[2 * t + 3]);
                }
            }
        }
        const double s = reduce_tile(v, lane);
        const int row = j0 + (lane >> 2);
        if ((lane & 1) == 0 && row < len)
            reinterpret_cast<double *>(part + off + j0)[lane >> 1] = s;
#pragma unroll
        for (int t = 0; t < kAdjTile; ++t) a[t] = an[t];
    }
}

template <int CH>
__global__ __launch_bounds__(64, CH == 8 ? 2 : CH == 1 ? 4 : 3) void k_legendre_adj(
    const PairDesc *__restrict__ pairs, LiveTab lt, int pblocks,
    const int *__restrict__ mval, const long long *__restrict__ moff, int nm, int nmpairs,
    int lmax, const double *__restrict__ A, const double2 *__restrict__ dt, DeltaLayout dl,
    double2 *__restrict__ part, long long nalm, int nmaps, int badm, int *__restrict__ bad)
{
    __shared__ double2 st[CH][64];
    // the same walk as the forward kernel's
    const int x = (int)(blockIdx.x % 8);
    const int w = (int)(blockIdx.x / 8);
    const int pb = w % pblocks;
    const int rest = w / pblocks;
    const int b = rest % nmaps;
    const int q = x + 8 * (rest / nmaps);
    if (q >= nmpairs) return;
    double2 *pp = part + ((long long)b * pblocks + pb) * nalm;
    for (int t = 0; t < 2; ++t) {
        const int i = (t == 0) ? q : nm - 1 - q;
        if (t == 1 && i == q) break;
        adj_one_m<CH>(pairs, lt, pb * CH, ((CIp)mval)[i], i, ((CLp)moff)[i], lmax, A,
                      dt + b * dl.map, dl, pp, st,
                      i < badm ? bad + ((long long)b * pblocks + pb) * badm + i : nullptr);
    }
}

// Sum of the ring blocks' partials, times c_lm; one thread per row of an m.
// Blocks that have no live row yet wrote nothing there.
template <int CH>
__global__ __launch_bounds__(256) void k_adj_reduce(
    const double2 *__restrict__ part, const double *__restrict__ cn, LiveTab lt,
    const int *__restrict__ mval, const long long *__restrict__ moff, int lmax,
    double *__restrict__ alm, long long nalm, int pblocks, int accumulate, int badm,
    const int *__restrict__ bad)
{
    const int i = blockIdx.y;
    const long long b = blockIdx.z;
    const int m = mval[i];
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= lmax - m + 1) return;
    const CIp jr = (CIp)(lt.jr + (long long)i * lt.nb);
    const long long e = moff[i] + j;
    // NaN if a ring of any block has an infinite or NaN Delta~ of this m (a
    // caller's), or of the set's first one (the analysis')
    const CIp bi = (CIp)(bad + b * pblocks * badm + (badm > 1 ? i : 0));
    int f = 0;
    for (int k = 0; k < pblocks; ++k) f |= bi[k * badm];
    double sr = f ? __builtin_nan("") : 0.0, si = sr;
    const double2 *p = part + b * pblocks * nalm + e;
    for (int k = 0; k < pblocks; ++k) {
        if (j >= adj_first_row<CH>(jr, k * CH)) {
            const double2 v = p[(long long)k * nalm];
            sr += v.x; si += v.y;
        }
    }
    const double c = cn[e];
    double2 *o = reinterpret_cast<double2 *>(alm) + b * nalm + e;
    const double2 v = make_double2(sr * c, m == 0 ? 0.0 : si * c);
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

__global__ __launch_bounds__(256) void k_batch_prescale(
    const BatchMap *__restrict__ maps, const double *const *__restrict__ alms,
    char *__restrict__ ws)
{
    const BatchMap &bm = maps[blockIdx.y];
    if ((int)blockIdx.x >= bm.nbad) return;
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    unsigned f = 0;
    if (e < bm.nalm) {
        const double2 *a = reinterpret_cast<const double2 *>(alms[blockIdx.y]);
        double2 v = a[e];
        const double c = bm.cn[e];
        v.x *= c;
        v.y = (e < bm.m0len) ? 0.0 : v.y * c;
        reinterpret_cast<double2 *>(ws + bm.ap_off)[e] = v;
        f = (isfinite(v.x) && isfinite(v.y)) ? 0u : 1u;
    }
    store_bad<1>(f, reinterpret_cast<unsigned char *>(ws + bm.bad_off) + blockIdx.x);
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
        load_chains(g, bm.pairs, tile.pblock * CH);
        const double2 *ap = reinterpret_cast<const double2 *>(ws + bm.ap_off);
        double2 *delta = reinterpret_cast<double2 *>(ws + bm.delta_off);
        const int q = tile.mpair;
        for (int u = 0; u < 2; ++u) {
            const int i = (u == 0) ? q : bm.nm - 1 - q;
            if (u == 1 && i == q) break;
            fwd_one_m<CH, 1>(g, bm.live, tile.pblock * CH, ((CIp)bm.mval)[i], i,
                             ((CLp)bm.moff)[i], bm.lmax, bm.A, ap, delta, bm.dl, false, bm.nbad,
                             reinterpret_cast<const unsigned char *>(ws + bm.bad_off));
        }
    }
}

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

// Blocks of 256 coefficients, and the bytes that note the infinite and NaN ones of
// every group of maps.
static int bad_blocks(const sht_plan_s *p) { return (int)((p->nalm + 255) / 256); }
size_t fwd_bad_bytes(const sht_plan_s *p)
{
    return p->precision == SHT_FP64 ? (size_t)p->nmaps * (size_t)bad_stride(bad_blocks(p)) : 0;
}

hipError_t launch_prescale(const sht_plan_s *p, const double *alm, double2 *ap,
                           unsigned char *bad, hipStream_t st)
{
    const long long m0len = (p->mval[0] == 0) ? (p->lmax + 1) : 0;
    const int nbad = bad_blocks(p);
    return for_map_groups(p, [&](int first, int groups, auto nb) {
        dim3 grid((unsigned)nbad, (unsigned)groups);
        hipLaunchKernelGGL(k_prescale<decltype(nb)::value>, grid, dim3(256), 0, st,
                           reinterpret_cast<const double2 *>(alm) + first * p->nalm, p->d_cn,
                           ap + first * p->nalm, p->nalm, m0len, nbad,
                           bad ? bad + first * bad_stride(nbad) : nullptr);
        return hipGetLastError();
    });
}

int fwd_pblocks(const sht_plan_s *p)
{
    const int per = 64 * p->fwd_chains;
    return (p->npairs + per - 1) / per;
}
int adj_pblocks(const sht_plan_s *p)
{
    const int per = 64 * p->adj_chains;
    return (p->npairs + per - 1) / per;
}

template <int NB>
static auto fwd_kernel(int chains) -> decltype(&k_legendre_fwd<1, NB>)
{
    return chains == 1   ? k_legendre_fwd<1, NB>
           : chains == 2 ? k_legendre_fwd<2, NB>
           : chains == 4 ? k_legendre_fwd<4, NB>
                         : nullptr;
}

hipError_t launch_legendre_fwd(const sht_plan_s *p, const double2 *ap, const unsigned char *bad,
                               double2 *delta, bool full, hipStream_t st)
{
    const int pblocks = fwd_pblocks(p);
    const int nmpairs = (p->nm + 1) / 2;
    const DeltaLayout dl = full ? delta_plain(p->nm, p->nrings) : delta_blocked(p->nm, p->nrings);
    return for_map_groups(p, [&](int first, int groups, auto nb) {
        const long long total = 8LL * ((nmpairs + 7) / 8) * pblocks * groups;
        if (total <= 0 || total > 0x7fffffffLL) return hipErrorInvalidConfiguration;
        const auto kern = fwd_kernel<decltype(nb)::value>(p->fwd_chains);
        if (!kern) return hipErrorInvalidValue;
        hipLaunchKernelGGL(kern, dim3((unsigned)total), dim3(64), 0, st, p->d_pairs, p->live,
                           pblocks, p->d_mval, p->d_moff, p->nm, nmpairs, p->lmax, p->d_A,
                           ap + first * p->nalm, p->nalm,
                           delta + first * dl.map, dl, groups, full ? 1 : 0, bad_blocks(p),
                           bad ? bad + first * bad_stride(bad_blocks(p)) : nullptr);
        return hipGetLastError();
    });
}

static size_t adj_sums(const sht_plan_s *p)
{
    return (size_t)p->nmaps * (size_t)adj_pblocks(p) * (size_t)p->nalm;
}
// the sums of the ring blocks, then one flag per (map, ring block, m)
size_t adj_part_bytes(const sht_plan_s *p)
{
    return adj_sums(p) * sizeof(double2) +
           (size_t)p->nmaps * (size_t)adj_pblocks(p) * (size_t)p->nm * sizeof(int);
}

template <int CH>
static hipError_t adj_launch(const sht_plan_s *p, const double2 *dt, bool plain, double2 *part,
                             double *alm, hipStream_t st, bool accumulate)
{
    const DeltaLayout dl = plain ? delta_plain(p->nm, p->nrings) : delta_blocked(p->nm, p->nrings);
    const int badm = plain ? p->nm : 1;   // flags per ring block: of every m, or of the first
    int *bad = reinterpret_cast<int *>(part + adj_sums(p));
    const int pblocks = adj_pblocks(p);
    const int nmpairs = (p->nm + 1) / 2;
    const long long total = 8LL * ((nmpairs + 7) / 8) * pblocks * p->nmaps;
    if (total <= 0 || total > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(k_legendre_adj<CH>, dim3((unsigned)total), dim3(64), 0, st, p->d_pairs,
                       p->live, pblocks, p->d_mval, p->d_moff, p->nm, nmpairs, p->lmax,
                       p->d_A, dt, dl, part, p->nalm, p->nmaps, badm, bad);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int longest = p->lmax - p->mval[0] + 1;
    dim3 grid((unsigned)((longest + 255) / 256), (unsigned)p->nm, (unsigned)p->nmaps);
    hipLaunchKernelGGL(k_adj_reduce<CH>, grid, dim3(256), 0, st, part, p->d_cn, p->live, p->d_mval,
                       p->d_moff, p->lmax, alm, p->nalm, pblocks, accumulate ? 1 : 0, badm, bad);
    return hipGetLastError();
}

hipError_t launch_legendre_adj_ws(const sht_plan_s *p, const double2 *dt, bool plain,
                                  double2 *part, double *alm, hipStream_t st, bool accumulate)
{
    switch (p->adj_chains) {
    case 1: return adj_launch<1>(p, dt, plain, part, alm, st, accumulate);
    case 2: return adj_launch<2>(p, dt, plain, part, alm, st, accumulate);
    case 8: return adj_launch<8>(p, dt, plain, part, alm, st, accumulate);
    default: return hipErrorInvalidValue;
    }
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
