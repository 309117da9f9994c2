// Per-ring Fourier step of alm2map and of its adjoint for gfx950: FP64,
// except the synthesis fast paths of the mixed forms (complex64 passes).
//
// Synthesis (Eq. Delta2map, Sec. 2.1, and the wrap rule of Sec. 2.2.2):
//     s_j = sum_{m=-mmax}^{mmax} Delta_m e^{i m (phi0 + 2 pi j / n)},  Delta_{-m} = conj(Delta_m).
// With D_m = Delta_m e^{i m phi0}, every mode is moved to bin m mod n:
//     F_k = sum_{m = k mod n} D_m + sum_{m >= 1, m = -k mod n} conj(D_m),
//     s_j = sum_{k<n} F_k e^{2 pi i j k / n}.
// F is Hermitian, so for even n the real inverse DFT is taken as one complex
// DFT of half length h = n/2:
//     Z_k = (F_k + conj F_{h-k}) + i e^{2 pi i k/n} (F_k - conj F_{h-k}),
//     z_j = sum_{k<h} Z_k e^{2 pi i j k/h},   s_2j = Re z_j,  s_2j+1 = Im z_j;
// odd n use a complex DFT of length n and keep the real part.
//
// Analysis (adjoint): G_k = sum_j g_j e^{-2 pi i j k / n} by the reverse
// construction, then Dt_m = c_m e^{-i m phi0} G_{m mod n} (c_0 = 1, c_m = 2).
//
// The whole ring lives in LDS, one workgroup to a ring and map (two maps in the
// mixed forms).  What each ring takes, in this order:
//  - fast path (k_ring_synth_fast, k_ring_anal_fast): even rings whose half
//    length is 7-smooth and at most 4096 (every HEALPix belt ring and the caps'
//    smooth ones).  A persistent kernel loads a ring's modes all at once (the
//    next ring's while the current one is transformed), folds them through a
//    padded LDS buffer and runs Stockham passes of radix 16, 8, 4, 2, 7, 5, 3
//    with the butterflies held in registers, the half-length pre-processing
//    fused into the first pass and the pixels stored from the last; the
//    analysis is the reverse, pixels into the first pass and modes out of LDS.
//    FP64 plans run it in complex128, and also take even rings of at most 64
//    points of half length on it, as a direct DFT.  The mixed forms, whose
//    Delta is complex64 with the maps of a ring contiguous, run the synthesis
//    in complex64, two maps of a ring per workgroup and one 16-byte load per
//    mode (the fold adds in FP64 either way).
//  - Bluestein fast path (k_ring_synth_blue and, in complex128 and also for
//    the analysis, k_ring_synth_blue64 / k_ring_anal_blue64): even rings whose
//    half length is even and not 7-smooth.  The even- and odd-indexed
//    convolutions run side by side in two buffers, with the chirps, the kernel
//    spectrum, the pre-processing and the stores inside the passes.
//  - everything else (odd lengths, half lengths above 4096 or odd and not
//    smooth; in the mixed forms' analysis all Bluestein rings, and for short
//    rings the smooth ones too; a caller's whole Delta on Bluestein rings):
//    size classes by FFT
//    length (up to 2048, 4096 and 8192 points) on 256-, 512- and 1024-thread
//    workgroups.  DFTs of 7-smooth length run as an in-place Stockham FFT
//    (radices 8, 4, 2, 3, 5 and 7; every pass loads its butterfly inputs into
//    registers, barriers, and stores); other lengths use Bluestein's chirp-z
//    algorithm with a 7-smooth convolution length whose kernel spectrum is
//    precomputed at plan time; an even length whose half is not 7-smooth is
//    split into the DFTs of its even- and odd-indexed inputs joined by one
//    radix-2 step.
// Twiddles come from per-length tables computed on the host in extended
// precision.
#include "sht_internal.h"

// Every fused multiply-add in this file is written out (fma, cmul): no
// contraction, so that all instantiations of the Fourier kernels (single and
// batched, any size class) round identically.
#pragma clang fp contract(off)

namespace sht {
namespace {


// Complex product with its roundings pinned (one product, then one fused
// multiply-add per component), so that every inlined copy of a kernel rounds
// alike whatever the compiler would otherwise contract.
__device__ inline double2 cmul(double2 a, double2 b)
{
    return make_double2(fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x));
}
__device__ inline double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ inline double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ inline double2 conjd(double2 a) { return make_double2(a.x, -a.y); }
// sign * i * a
__device__ inline double2 muli(double2 a, int sign)
{
    return sign > 0 ? make_double2(-a.y, a.x) : make_double2(a.y, -a.x);
}

// The same operations on complex64, for the FP32 Fourier passes of the mixed
// forms' fast path.
__device__ inline float2 cmul(float2 a, float2 b)
{
    return make_float2(fmaf(a.x, b.x, -(a.y * b.y)), fmaf(a.x, b.y, a.y * b.x));
}
__device__ inline float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ inline float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ inline float2 conjd(float2 a) { return make_float2(a.x, -a.y); }
__device__ inline float2 muli(float2 a, int sign)
{
    return sign > 0 ? make_float2(-a.y, a.x) : make_float2(a.y, -a.x);
}

// Complex element type C from real parts, and conversions between the two
// precisions (rounded once).
template <typename C> __device__ inline C cplx(double x, double y);
template <> __device__ inline double2 cplx<double2>(double x, double y) { return make_double2(x, y); }
template <> __device__ inline float2 cplx<float2>(double x, double y)
{
    return make_float2((float)x, (float)y);
}
template <typename C> __device__ inline C cvt(double2 v) { return cplx<C>(v.x, v.y); }
__device__ inline double2 todbl(double2 v) { return v; }
__device__ inline double2 todbl(float2 v) { return make_double2((double)v.x, (double)v.y); }

// cos / sin of 2 pi q / R (correctly rounded)
template <int R> struct Roots;
template <> struct Roots<3> {
    static constexpr double c[3] = {0x1p+0, -0x1p-1, -0x1p-1};
    static constexpr double s[3] = {0.0, 0x1.bb67ae8584caap-1, -0x1.bb67ae8584caap-1};
};
template <> struct Roots<5> {
    static constexpr double c[5] = {0x1p+0, 0x1.3c6ef372fe950p-2, -0x1.9e3779b97f4a8p-1,
                                    -0x1.9e3779b97f4a8p-1, 0x1.3c6ef372fe950p-2};
    static constexpr double s[5] = {0.0, 0x1.e6f0e134454ffp-1, 0x1.2cf2304755a5ep-1,
                                    -0x1.2cf2304755a5ep-1, -0x1.e6f0e134454ffp-1};
};
template <> struct Roots<7> {
    static constexpr double c[7] = {0x1p+0, 0x1.3f3a0e28bedd1p-1, -0x1.c7b90e3024582p-3,
                                    -0x1.cd4bca9cb5c71p-1, -0x1.cd4bca9cb5c71p-1,
                                    -0x1.c7b90e3024582p-3, 0x1.3f3a0e28bedd1p-1};
    static constexpr double s[7] = {0.0, 0x1.904c37505de4bp-1, 0x1.f329c0558e969p-1,
                                    0x1.bc4c04d71abc1p-2, -0x1.bc4c04d71abc1p-2,
                                    -0x1.f329c0558e969p-1, -0x1.904c37505de4bp-1};
};

// y_k = sum_r v_r e^{sign 2 pi i r k / R}
__device__ inline double fmaS(double a, double b, double c) { return fma(a, b, c); }
__device__ inline float fmaS(float a, float b, float c) { return fmaf(a, b, c); }

template <int R, typename C>
__device__ inline void small_dft(C (&v)[R], int sign)
{
    typedef decltype(C::x) S;
    if constexpr (R == 2) {
        const C a = v[0], b = v[1];
        v[0] = cadd(a, b);
        v[1] = csub(a, b);
    } else if constexpr (R == 4) {
        const C s02 = cadd(v[0], v[2]), d02 = csub(v[0], v[2]);
        const C s13 = cadd(v[1], v[3]), d13 = muli(csub(v[1], v[3]), sign);
        v[0] = cadd(s02, s13);
        v[2] = csub(s02, s13);
        v[1] = cadd(d02, d13);
        v[3] = csub(d02, d13);
    } else if constexpr (R == 16) {
        // 16 = 4 x 4: r = 4a + b, k = c + 4d, w^(rk) = w4^(ac) w16^(bc) w4^(bd)
        C u[4][4];   // u[b][c]
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            C t[4] = {v[b], v[4 + b], v[8 + b], v[12 + b]};
            small_dft<4, C>(t, sign);
#pragma unroll
            for (int c = 0; c < 4; ++c) u[b][c] = t[c];
        }
        constexpr S c1 = (S) 0x1.d906bcf328d46p-1;  // cos(pi/8), correctly rounded
        constexpr S s1 = (S) 0x1.87de2a6aea963p-2;  // sin(pi/8)
        constexpr S hh = (S) 0x1.6a09e667f3bcdp-1;  // 1/sqrt(2)
        // w16^e = (cos, sign sin) of 2 pi e / 16 for e = b c, b, c in 1..3
        const S sg = (S)sign;
        u[1][1] = cmul(u[1][1], cplx<C>(c1, sg * s1));
        u[1][2] = cmul(u[1][2], cplx<C>(hh, sg * hh));
        u[1][3] = cmul(u[1][3], cplx<C>(s1, sg * c1));
        u[2][1] = cmul(u[2][1], cplx<C>(hh, sg * hh));
        u[2][2] = muli(u[2][2], sign);
        u[2][3] = cmul(u[2][3], cplx<C>(-hh, sg * hh));
        u[3][1] = cmul(u[3][1], cplx<C>(s1, sg * c1));
        u[3][2] = cmul(u[3][2], cplx<C>(-hh, sg * hh));
        u[3][3] = cmul(u[3][3], cplx<C>(-c1, -sg * s1));
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            C t[4] = {u[0][c], u[1][c], u[2][c], u[3][c]};
            small_dft<4, C>(t, sign);
#pragma unroll
            for (int d = 0; d < 4; ++d) v[c + 4 * d] = t[d];
        }
    } else if constexpr (R == 8) {
        // two radix-4 DFTs of the even and odd inputs, combined with w8^k
        C e[4] = {v[0], v[2], v[4], v[6]};
        C o[4] = {v[1], v[3], v[5], v[7]};
        small_dft<4, C>(e, sign);
        small_dft<4, C>(o, sign);
        constexpr S h = (S)0x1.6a09e667f3bcdp-1;  // 1/sqrt(2), correctly rounded
        // w8 = e^{sign i pi/4}: w8^1 o1, w8^2 o2 = sign i o2, w8^3 o3
        const C t1 = cplx<C>(h * (o[1].x - sign * o[1].y), h * (o[1].y + sign * o[1].x));
        const C t2 = muli(o[2], sign);
        const C t3 = cplx<C>(-h * (o[3].x + sign * o[3].y), h * (sign * o[3].x - o[3].y));
        v[0] = cadd(e[0], o[0]);
        v[4] = csub(e[0], o[0]);
        v[1] = cadd(e[1], t1);
        v[5] = csub(e[1], t1);
        v[2] = cadd(e[2], t2);
        v[6] = csub(e[2], t2);
        v[3] = cadd(e[3], t3);
        v[7] = csub(e[3], t3);
    } else {
        // odd R: pair r with R - r
        C sp[R / 2], dm[R / 2];
#pragma unroll
        for (int r = 1; r <= R / 2; ++r) {
            sp[r - 1] = cadd(v[r], v[R - r]);
            dm[r - 1] = csub(v[r], v[R - r]);
        }
        C y[R];
        C y0 = v[0];
#pragma unroll
        for (int r = 0; r < R / 2; ++r) y0 = cadd(y0, sp[r]);
        y[0] = y0;
#pragma unroll
        for (int k = 1; k < R; ++k) {
            S ar = v[0].x, ai = v[0].y, br = 0, bi = 0;
#pragma unroll
            for (int r = 1; r <= R / 2; ++r) {
                const S c = (S)Roots<R>::c[(r * k) % R];
                const S s = (S)Roots<R>::s[(r * k) % R];
                ar = fmaS(sp[r - 1].x, c, ar);
                ai = fmaS(sp[r - 1].y, c, ai);
                br = fmaS(dm[r - 1].x, s, br);
                bi = fmaS(dm[r - 1].y, s, bi);
            }
            // + sign * i * (b)
            y[k] = sign > 0 ? cplx<C>(ar - bi, ai + br) : cplx<C>(ar + bi, ai - br);
        }
#pragma unroll
        for (int k = 0; k < R; ++k) v[k] = y[k];
    }
}

// Twiddles e^{+2 pi i t / L} (t < L <= 16384) from a two-level table in LDS:
// T[b] = w^b for b < 64 and T[64 + a] = w^(64 a), so w^t = T[64 + t/64] T[t % 64]
// (within 2 ulp; T[64] = 1 exactly).  Filled from the plan's full table `tab`
// (entry t at tab[t]) at the start of a workgroup, so that the FFT passes
// never wait on global memory.
constexpr int kTwEntries = 64 + 256;

template <int NT, typename C>
__device__ __attribute__((always_inline)) inline void load_tw(C *T, const double2 *__restrict__ tab,
                                                              int L)
{
    const int n1 = (L + 63) >> 6;
    for (int e = threadIdx.x; e < 64 + n1; e += NT) {
        const int t = (e < 64) ? e : 64 * (e - 64);
        T[e] = (t < L) ? cvt<C>(tab[t]) : cplx<C>(1.0, 0.0);
    }
}

// The same from a complex64 copy of the table.
template <int NT>
__device__ __attribute__((always_inline)) inline void load_tw(float2 *T,
                                                              const float2 *__restrict__ tab,
                                                              int L)
{
    const int n1 = (L + 63) >> 6;
    for (int e = threadIdx.x; e < 64 + n1; e += NT) {
        const int t = (e < 64) ? e : 64 * (e - 64);
        T[e] = (t < L) ? tab[t] : make_float2(1.0f, 0.0f);
    }
}

template <typename C>
__device__ inline C tw_at(const C *T, int t)
{
    return cmul(T[64 + (t >> 6)], T[t & 63]);
}

// One Stockham pass of radix R over n <= MAXN points in LDS.  T is the LDS
// table of e^{+2 pi i t / L} with L = n * tws.  j / Ns is taken as
// umulhi(j, ceil(2^32 / Ns)), which is exact for j, Ns < 2^13.
template <int R, int NT, int MAXN>
__device__ __attribute__((always_inline)) inline void fft_pass(double2 *buf, int n, int Ns, int sign, const double2 *T,
                         int tws)
{
    constexpr int MAXQ = (MAXN / R + NT - 1) / NT;
    const int nb = n / R;
    const int tstep0 = (n / (Ns * R)) * tws;
    const unsigned magic = (unsigned)((0x100000000ull + (unsigned)Ns - 1) / (unsigned)Ns);
    double2 v[MAXQ][R];
#pragma unroll
    for (int q = 0; q < MAXQ; ++q) {
        const int j = threadIdx.x + q * NT;
        if (j < nb) {
            const int jq = (Ns == 1) ? j : (int)__umulhi((unsigned)j, magic);
            const int k = j - jq * Ns;
            const int ts = tstep0 * k;
            // twiddles w^r, r = 1..R-1, as powers of one table entry w
            double2 w1 = make_double2(1.0, 0.0);
            if (ts != 0) {
                w1 = tw_at(T, ts);
                if (sign < 0) w1.y = -w1.y;
            }
            double2 wr = w1;
            v[q][0] = buf[j];
#pragma unroll
            for (int r = 1; r < R; ++r) {
                const double2 x = buf[j + r * nb];
                v[q][r] = (ts != 0) ? cmul(x, wr) : x;
                wr = cmul(wr, w1);
            }
            small_dft<R>(v[q], sign);
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < MAXQ; ++q) {
        const int j = threadIdx.x + q * NT;
        if (j < nb) {
            const int jq = (Ns == 1) ? j : (int)__umulhi((unsigned)j, magic);
            const int k = j - jq * Ns;
            const int base = jq * Ns * R + k;
#pragma unroll
            for (int r = 0; r < R; ++r) buf[base + r * Ns] = v[q][r];
        }
    }
    __syncthreads();
}

// In-place DFT of 7-smooth length n <= MAXN:
// buf_k <- sum_j buf_j e^{sign 2 pi i j k / n}.
template <int NT, int MAXN>
__device__ __attribute__((always_inline)) inline void fft_lds(double2 *buf, int n, int sign, const double2 *T, int tws)
{
    int Ns = 1, rem = n;
    while (rem > 1) {
        if (rem % 8 == 0) {
            fft_pass<8, NT, MAXN>(buf, n, Ns, sign, T, tws); Ns *= 8; rem /= 8;
        } else if (rem % 4 == 0) {
            fft_pass<4, NT, MAXN>(buf, n, Ns, sign, T, tws); Ns *= 4; rem /= 4;
        } else if (rem % 2 == 0) {
            fft_pass<2, NT, MAXN>(buf, n, Ns, sign, T, tws); Ns *= 2; rem /= 2;
        } else if (rem % 3 == 0) {
            fft_pass<3, NT, MAXN>(buf, n, Ns, sign, T, tws); Ns *= 3; rem /= 3;
        } else if (rem % 5 == 0) {
            fft_pass<5, NT, MAXN>(buf, n, Ns, sign, T, tws); Ns *= 5; rem /= 5;
        } else {
            fft_pass<7, NT, MAXN>(buf, n, Ns, sign, T, tws); Ns *= 7; rem /= 7;
        }
    }
}

// In-place DFT of any length len by Bluestein's algorithm:
// e^{i 2 pi jk/len} = c_j c_k conj(c_{j-k}), c_k = e^{i pi k^2 / len}, as a
// cyclic convolution of 7-smooth length nb >= 2 len - 1.
// ch = this thread's chirps c_k, k = tid + q NT (loaded ahead by the caller),
// TB = LDS table of e^{2 pi i k / nb}, bq = DFT^-(conj c, wrapped) / nb.
// A sign -1 transform is conj(DFT^+(conj x)).
// REG: the chirps are held in registers from the start of the workgroup
// (their load latency overlaps the fold), else read where used.
template <int NT, int MAXN, bool REG>
struct Chirps {
    static constexpr int Q = (MAXN / 2 + NT - 1) / NT;  // len <= (nb + 1) / 2 <= MAXN / 2
    double2 c[REG ? Q : 1];
    const double2 *p;
    __device__ double2 get(int q, int k) const { return REG ? c[REG ? q : 0] : p[k]; }
};

template <int NT, int MAXN, bool REG>
__device__ __attribute__((always_inline)) inline void load_chirps(Chirps<NT, MAXN, REG> &ch,
                                                                  const double2 *__restrict__ chirp,
                                                                  int len)
{
    ch.p = chirp;
    if (REG) {
#pragma unroll
        for (int q = 0; q < Chirps<NT, MAXN, REG>::Q; ++q) {
            const int k = threadIdx.x + q * NT;
            ch.c[REG ? q : 0] = (k < len) ? chirp[k] : make_double2(0.0, 0.0);
        }
    }
}

template <int NT, int MAXN, bool REG>
__device__ __attribute__((always_inline)) inline void bluestein_lds(double2 *buf, int len, int nb, int sign,
                              const Chirps<NT, MAXN, REG> &ch, const double2 *TB,
                              const double2 *__restrict__ bq)
{
    constexpr int QB = MAXN / NT;
#pragma unroll
    for (int q = 0; q < QB; ++q) {
        const int k = threadIdx.x + q * NT;
        if (k < nb) {
            if (q < Chirps<NT, MAXN, REG>::Q && k < len) {
                double2 x = buf[k];
                if (sign < 0) x.y = -x.y;
                buf[k] = cmul(x, ch.get(q < Chirps<NT, MAXN, REG>::Q ? q : 0, k));
            } else {
                buf[k] = make_double2(0.0, 0.0);
            }
        }
    }
    __syncthreads();
    fft_lds<NT, MAXN>(buf, nb, -1, TB, 1);
#pragma unroll
    for (int q = 0; q < QB; ++q) {
        const int k = threadIdx.x + q * NT;
        if (k < nb) buf[k] = cmul(buf[k], bq[k]);
    }
    __syncthreads();
    fft_lds<NT, MAXN>(buf, nb, +1, TB, 1);
#pragma unroll
    for (int q = 0; q < Chirps<NT, MAXN, REG>::Q; ++q) {
        const int j = threadIdx.x + q * NT;
        if (j < len) {
            double2 z = cmul(buf[j], ch.get(q, j));
            if (sign < 0) z.y = -z.y;
            buf[j] = z;
        }
    }
    __syncthreads();
}

// LDS tables of a ring's Fourier step: TW for e^{2 pi i k / n} (n-point
// roots: the half-length FFT and its pre/post twiddles), TB for the
// Bluestein length.
struct RingTables {
    double2 *TW;
    double2 *TB;
};

template <int NT, int MAXN, bool REG>
__device__ __attribute__((always_inline)) inline void ring_tables_load(const RingTables &rt,
                                                                       const RingDesc &d,
                                                                       const double2 *__restrict__ pool,
                                                                       Chirps<NT, MAXN, REG> &ch)
{
    load_tw<NT>(rt.TW, pool + d.tw, d.n);
    if (d.nb != 0) {
        load_tw<NT>(rt.TB, pool + d.twb, d.nb);
        load_chirps<NT, MAXN, REG>(ch, pool + d.tch, d.half ? d.clen / 2 : d.clen);
    }
}

// DFT of even length clen = 2 len whose half length is not 7-smooth:
// with E = DFT_len(x_{2j}) and O = DFT_len(x_{2j+1}) (Bluestein each, one
// after the other in the same LDS buffer), X_j = E_j + w^j O_j and
// X_{j+len} = E_j - w^j O_j, w = e^{sign 2 pi i / clen}.  The ring is even,
// so TW holds the n-th roots with n = 2 clen: w^j = TW(2 j).  PRIV: the
// half kept across each Bluestein transform lives in private memory instead
// of registers (for kernels whose register budget is already spent).
template <int NT, int MAXN, bool REG, bool PRIV>
__device__ __attribute__((always_inline)) inline void split_bluestein(
    double2 *buf, const RingDesc &d, int sign, const double2 *__restrict__ pool,
    const RingTables &rt, const Chirps<NT, MAXN, REG> &ch)
{
    constexpr int QH = (MAXN / 2 + NT - 1) / NT;
    const int len = d.clen / 2;
    const int tid = threadIdx.x;
    double2 keep[QH], odd[QH];
    int zq = 0;   // an opaque zero index keeps the arrays out of registers
    if constexpr (PRIV) asm volatile("" : "+s"(zq));
#pragma unroll
    for (int q = 0; q < QH; ++q) {
        const int j = tid + q * NT;
        if (j < len) {
            keep[q ^ zq] = buf[2 * j];
            odd[q ^ zq] = buf[2 * j + 1];
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < QH; ++q) {
        const int j = tid + q * NT;
        if (j < len) buf[j] = keep[q ^ zq];
    }
    __syncthreads();
    bluestein_lds<NT, MAXN, REG>(buf, len, d.nb, sign, ch, rt.TB, pool + d.bq);
#pragma unroll
    for (int q = 0; q < QH; ++q) {
        const int j = tid + q * NT;
        if (j < len) keep[q ^ zq] = buf[j];   // E_j
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < QH; ++q) {
        const int j = tid + q * NT;
        if (j < len) buf[j] = odd[q ^ zq];
    }
    __syncthreads();
    bluestein_lds<NT, MAXN, REG>(buf, len, d.nb, sign, ch, rt.TB, pool + d.bq);
#pragma unroll
    for (int q = 0; q < QH; ++q) {
        const int j = tid + q * NT;
        if (j < len) {
            double2 w = tw_at(rt.TW, 2 * j);
            if (sign < 0) w.y = -w.y;
            const double2 t = cmul(w, buf[j]);
            const double2 e = keep[q ^ zq];
            buf[j] = cadd(e, t);
            buf[j + len] = csub(e, t);
        }
    }
    __syncthreads();
}

template <int NT, int MAXN, bool REG, bool PRIV = false>
__device__ __attribute__((always_inline)) inline void ring_dft(double2 *buf, const RingDesc &d, int sign,
                                const double2 *__restrict__ pool, const RingTables &rt,
                                const Chirps<NT, MAXN, REG> &ch)
{
    if (d.nb == 0) {
        fft_lds<NT, MAXN>(buf, d.clen, sign, rt.TW, (d.n % 2 == 0) ? 2 : 1);
    } else if (d.half) {
        split_bluestein<NT, MAXN, REG, PRIV>(buf, d, sign, pool, rt, ch);
    } else {
        bluestein_lds<NT, MAXN, REG>(buf, d.clen, d.nb, sign, ch, rt.TB, pool + d.bq);
    }
}

// Block id -> logical id so that consecutive logical ids run on one XCD
// (workgroups are dealt round-robin over the 8 XCDs).
__device__ inline int xcd_logical(int b, int total)
{
    const int x = b % 8, i = b / 8, q = total / 8, r = total % 8;
    return x * q + (x < r ? x : r) + i;
}

// Work item -> (index in the class's ring list, map), so that the
// workgroups running together read Delta entries that share cache lines and
// DRAM pages: for [map][m][ring] Delta map by map, ring by ring
// (neighbouring rings of one map; measured faster than grouping a few rings'
// items of all maps together, which would keep each ring's tables in L2 but
// spreads the Delta reads over all maps); for Delta with the maps of a ring contiguous, ring by
// ring, map by map (all maps of one ring).
template <bool RM>
__device__ inline void ring_item(long long it, int count, int nmaps, int &i, int &b)
{
    if (RM) {
        i = (int)(it / nmaps);
        b = (int)(it - (long long)i * nmaps);
    } else {
        b = (int)(it / count);
        i = (int)(it - (long long)b * count);
    }
}

// The persistent kernels' share of XCD x (workgroups are dealt to the 8 XCDs
// round-robin): items [lo, hi) of its own numbering, item k -> (i, b).  Map
// by map: a contiguous eighth of all items.  Ring by ring: every eighth group
// of 2^shift rings (the class's rings are sorted by length, so every XCD gets
// rings of every length), all maps of a ring together; the groups hold the
// rings that share lines of Delta.
template <bool RM>
__device__ inline void xcd_share(int count, int nmaps, int x, int shift, long long &lo,
                                 long long &hi)
{
    if (RM) {
        // groups of 2^shift rings, dealt to the XCDs in turn
        const int g = 1 << shift, all = count >> (shift + 3);
        const int rest = count - (all << (shift + 3)) - (x << shift);
        lo = 0;
        hi = (long long)((all << shift) + (rest < 0 ? 0 : rest < g ? rest : g)) * nmaps;
    } else {
        const long long total = (long long)count * nmaps;
        lo = total * x / 8;
        hi = total * (x + 1) / 8;
    }
}

template <bool RM>
__device__ inline void xcd_item(long long k, int count, int nmaps, int x, int shift, int &i, int &b)
{
    if (RM) {
        const int q = (int)(k / nmaps);
        i = ((((q >> shift) << 3) + x) << shift) + (q & ((1 << shift) - 1));
        b = (int)(k - (long long)q * nmaps);
    } else {
        ring_item<false>(k, count, nmaps, i, b);
    }
}

// complex64 Delta (the mixed forms') has the maps of a ring contiguous: ring by ring
template <typename DT> struct RingMajor {
    static constexpr bool value = false;
};
template <> struct RingMajor<float2> {
    static constexpr bool value = true;
};

// Delta_m for mode m of a ring (zero for m outside the set); the ring's modes
// are `dstride` entries apart (DeltaLayout).  DT is the stored element: complex128, or complex64 from the mixed-precision
// Legendre stage (widened exactly).
__device__ inline double2 widen(double2 v) { return v; }
__device__ inline double2 widen(float2 v) { return make_double2((double)v.x, (double)v.y); }

template <typename DT>
__device__ inline double2 load_mode(const DT *__restrict__ drow, long long dstride,
                                    const int *__restrict__ minv, int mcontig, int m)
{
    const int i = mcontig ? m : minv[m];
    return (i >= 0) ? widen(drow[(long long)i * dstride]) : make_double2(0.0, 0.0);
}

// Modes of a ring: the Legendre stage of the plan leaves the m beyond the
// ring's mlive out (they are dead there, live.hip), so its rings fold
// m <= mlive (mfull < 0).  A caller's Delta has all of them: m <= mfull.
template <typename DT> __device__ inline int ring_live(const RingDesc &d) { return d.mlive; }
template <> __device__ inline int ring_live<float2>(const RingDesc &d) { return d.mlive32; }
template <typename DT = double2>
__device__ inline int ring_mmax(const RingDesc &d, int mfull)
{
    return mfull < 0 ? ring_live<DT>(d) : mfull;
}

// Synthesis: one workgroup per (ring of this size class, map).  LDS: the
// spectrum / FFT buffer, the twiddle tables and the alias staging slots
// (RingLds).
// Synthesis of one ring: drow = its Delta_m row, out = its first pixel.
// Padded LDS indexing of the fast path's spectrum / FFT buffer.
struct PadIdx {   // one spare entry per 16 (bank-conflict-free strided stores)
    __device__ static int at(int i) { return i + (i >> 4); }
};

// Fold a ring's modes into its spectrum F_k, k = 0..kmax (Eq. Delta2map with
// the wrap rule of Sec. 2.2.2; ends with a barrier).  drow = the ring's
// Delta_m row, the i-th m of the set at drow[i dstride].
template <int NT, typename DT>
__device__ __attribute__((always_inline)) inline void fold_ring(double2 *buf, const RingDesc &d,
                                                                const DT *__restrict__ drow,
                                                                long long dstride,
                                                                const int *__restrict__ minv,
                                                                int mcontig, int mmax)
{
    const int n = d.n;
    const bool even = (n % 2) == 0;
    const int h = n / 2;
    const int kmax = even ? h : n - 1;
    const int tid = threadIdx.x;
    // ---- fold the modes into F_k, k = 0..kmax (Sec. 2.2.2 wrap rule).
    // Phases e^{i m phi0}: one sincos per thread for its first mode and one
    // for the stride NT, then a complex multiply per further mode (a few ulp).
    constexpr int kBatch = 8;
    double2 step;   // e^{i NT phi0}
    double2 ph;     // e^{i tid phi0}
    {
        double sn, cs;
        sincos((double)NT * d.phi0, &sn, &cs);
        step = make_double2(cs, sn);
        sincos((double)tid * d.phi0, &sn, &cs);
        ph = make_double2(cs, sn);
    }
    if (n > mmax) {
        // each bin gets at most one direct mode m = k and one mirrored mode
        // m = n - k: F_k = e^{i k phi0} (D_k + e^{-i n phi0} conj(D_{n-k}))
        double2 cn;
        {
            double sn, cs;
            sincos((double)n * d.phi0, &sn, &cs);
            cn = make_double2(cs, -sn);
        }
        const int kdir = min(kmax, mmax);
        for (int k0 = 0; k0 <= kmax; k0 += kBatch * NT) {
            double2 raw[kBatch], rawc[kBatch];
#pragma unroll
            for (int q = 0; q < kBatch; ++q) {
                const int k = k0 + q * NT + tid;
                raw[q] = (k <= kdir) ? load_mode(drow, dstride, minv, mcontig, k) : make_double2(0.0, 0.0);
                rawc[q] = (k >= 1 && k <= kmax && n - k <= mmax)
                              ? load_mode(drow, dstride, minv, mcontig, n - k) : make_double2(0.0, 0.0);
            }
#pragma unroll
            for (int q = 0; q < kBatch; ++q) {
                const int k = k0 + q * NT + tid;
                if (k <= kmax) {
                    double2 D = raw[q];
                    if (k == 0) D.y = 0.0;
                    D = cadd(D, cmul(cn, conjd(rawc[q])));
                    buf[k] = cmul(ph, D);
                }
                ph = cmul(ph, step);
            }
        }
    } else {
        // wrap-around (n <= mmax): bin k gathers its aliases m = k + j n and
        // m = j n - k directly.  With w = e^{i n phi0},
        //   F_k = e^{i k phi0} (sum_j Delta_{k+jn} w^j + sum_{j>=1} conj(Delta_{jn-k}) conj(w^j)).
        // Few bins (small rings): G = NT / B threads share a bin, each taking
        // every G-th alias, and the G partial sums are staged in the spectrum
        // buffer itself (the class layout gives it at least NT entries when
        // some ring has fewer bins than threads) and added in a fixed order.
        // G depends on the ring and NT only, so every launch of the ring
        // rounds alike.  The aliases are fetched two at a time.
        const int B = kmax + 1;
        const int G = (B < NT) ? NT / B : 1;
        double2 step;    // e^{i NT phi0}
        {
            double sn, cs;
            sincos((double)NT * d.phi0, &sn, &cs);
            step = make_double2(cs, sn);
        }
        const int kk = (G > 1) ? tid % B : tid;
        const int g = (G > 1) ? tid / B : 0;
        double2 stepG;   // w^G
        {
            double sn, cs;
            sincos((double)n * (double)G * d.phi0, &sn, &cs);
            stepG = make_double2(cs, sn);
        }
        double2 phb;     // e^{i k phi0} for this thread's first bin
        {
            double sn, cs;
            sincos((double)kk * d.phi0, &sn, &cs);
            phb = make_double2(cs, sn);
        }
        constexpr int U = 2;
        for (int k = kk; k <= kmax && g < G; k += NT) {
            const int jmax = (mmax + k) / n;   // last alias with j n - k <= mmax
            double sr = 0.0, si = 0.0;
            int c = 0;
            double2 wj = make_double2(1.0, 0.0);
            for (int j0 = g; j0 <= jmax; j0 += U * G) {
                double2 Dd[U], Dm[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int j = j0 + u * G;
                    const int md = k + j * n, mc = j * n - k;
                    Dd[u] = make_double2(0.0, 0.0);
                    Dm[u] = make_double2(0.0, 0.0);
                    if (j <= jmax) {
                        if (md <= mmax) Dd[u] = load_mode(drow, dstride, minv, mcontig, md);
                        if (j >= 1) Dm[u] = load_mode(drow, dstride, minv, mcontig, mc);
                    }
                    if (md == 0) Dd[u].y = 0.0;
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int j = j0 + u * G;
                    if (j <= jmax) {
                        if ((c & 31) == 0) {   // re-seed w^j every 32 aliases
                            double sn, cs;
                            sincos((double)j * (double)n * d.phi0, &sn, &cs);
                            wj = make_double2(cs, sn);
                        }
                        const double2 v = cmul(Dd[u], wj);
                        sr += v.x; si += v.y;
                        const double2 vm = cmul(conjd(Dm[u]), conjd(wj));
                        sr += vm.x; si += vm.y;
                        wj = cmul(wj, stepG);
                        ++c;
                    }
                }
            }
            if (G > 1) {
                buf[g * B + k] = make_double2(sr, si);
            } else {
                buf[k] = cmul(phb, make_double2(sr, si));
                phb = cmul(phb, step);
            }
        }
        if (G > 1) {
            __syncthreads();
            // column k of the staged partials is read and then overwritten
            // (entry 0) by thread k alone
            if (tid < B) {
                double sr = 0.0, si = 0.0;
                for (int q = 0; q < G; ++q) {
                    const double2 v = buf[q * B + tid];
                    sr += v.x; si += v.y;
                }
                buf[tid] = cmul(phb, make_double2(sr, si));
            }
        }
    }
    __syncthreads();
}

template <int NT, int MAXN, bool REG, bool PRIV, typename DT>
__device__ __attribute__((always_inline)) inline void synth_ring(double2 *buf, const RingTables &rt, const RingDesc &d,
                           const double2 *__restrict__ pool, const DT *__restrict__ drow,
                           long long dstride, const int *__restrict__ minv, int mcontig, int mmax,
                           double *__restrict__ out)
{
    Chirps<NT, MAXN, REG> ch;
    ring_tables_load<NT, MAXN, REG>(rt, d, pool, ch);
    const int n = d.n;
    const bool even = (n % 2) == 0;
    const int h = n / 2;
    const int tid = threadIdx.x;
    fold_ring<NT>(buf, d, drow, dstride, minv, mcontig, mmax);
    if (even) {
        for (int k = tid; k <= h / 2; k += NT) {
            const int k2 = h - k;
            const double2 Fk = buf[k], Fk2 = buf[k2];
            const double2 e1 = cadd(Fk, conjd(Fk2)), o1 = csub(Fk, conjd(Fk2));
            const double2 Zk = cadd(e1, muli(cmul(tw_at(rt.TW, k), o1), +1));
            const double2 e2 = cadd(Fk2, conjd(Fk)), o2 = csub(Fk2, conjd(Fk));
            const double2 Zk2 = cadd(e2, muli(cmul(tw_at(rt.TW, k2), o2), +1));
            buf[k] = Zk;
            if (k2 != k) buf[k2] = Zk2;
        }
        __syncthreads();
        ring_dft<NT, MAXN, REG, PRIV>(buf, d, +1, pool, rt, ch);
        if ((reinterpret_cast<uintptr_t>(out) & 15) == 0) {
            double2 *o2 = reinterpret_cast<double2 *>(out);
            for (int j = tid; j < h; j += NT) o2[j] = buf[j];
        } else {
            for (int j = tid; j < h; j += NT) {
                const double2 z = buf[j];
                out[2 * j] = z.x;
                out[2 * j + 1] = z.y;
            }
        }
    } else {
        ring_dft<NT, MAXN, REG, PRIV>(buf, d, +1, pool, rt, ch);
        for (int j = tid; j < n; j += NT) out[j] = buf[j].x;
    }
}


// ---------------------------------------------------------------------------
// Fast path of the synthesis: even rings whose half length h is 7-smooth and
// at most kFastMaxH.  The spectrum sits in a padded LDS buffer (PadIdx), each
// Stockham pass holds its butterflies in registers (radix 16, 8, 4, 2, 7, 5,
// 3 from the ring's pass list), the half-length pre-processing Z_k is formed
// while the first pass loads its inputs, and the last pass writes the pixels
// straight from registers: per ring one fold, one barrier pair per inner
// pass and no other LDS round trip.
//
// One pass of radix R over the h-point buffer (input index j + r h/R,
// output index (j / Ns) Ns R + j % Ns + r Ns).  T: the ring's n-th roots.
// tid: the thread's place among the NT that share the buffer; store: the last
// pass writes the pixels (not for a map that is not there).
template <int R, int NT, typename C>
__device__ __attribute__((always_inline)) inline void fast_pass(C *buf, const C *T,
                                                                int h, int Ns, bool first,
                                                                bool last, double *__restrict__ out,
                                                                int tid, bool store)
{
    constexpr int MAXQ = fast_maxq(R);   // the plan admits h / R <= MAXQ * kFastThreads
    const int nb = h / R;
    const int tstep0 = (h / (Ns * R)) * 2;   // T holds the roots of n = 2 h
    const unsigned magic = (unsigned)((0x100000000ull + (unsigned)Ns - 1) / (unsigned)Ns);
    // an opaque copy of the thread index: the passes run in a loop over the
    // ring's radix list, and address arithmetic hoisted out of every radix's
    // case would stay live across all of them
    asm volatile("" : "+v"(tid));
    C v[MAXQ][R];
#pragma unroll
    for (int q = 0; q < MAXQ; ++q) {
        const int j = tid + q * NT;
        if (j < nb) {
            if (first) {
                // Z_k = (F_k + conj F_{h-k}) + i e^{2 pi i k/n} (F_k - conj F_{h-k})
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int k = j + r * nb;
                    const C Fk = buf[PadIdx::at(k)], Fk2 = buf[PadIdx::at(h - k)];
                    const C e1 = cadd(Fk, conjd(Fk2)), o1 = csub(Fk, conjd(Fk2));
                    v[q][r] = cadd(e1, muli(cmul(tw_at(T, k), o1), +1));
                }
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r) v[q][r] = buf[PadIdx::at(j + r * nb)];
            }
            if (Ns > 1) {
                const int jq = (int)__umulhi((unsigned)j, magic);
                const int ts = tstep0 * (j - jq * Ns);
                if (ts != 0) {
                    const C w1 = tw_at(T, ts);
                    C wr = w1;
#pragma unroll
                    for (int r = 1; r < R; ++r) {
                        v[q][r] = cmul(v[q][r], wr);
                        wr = cmul(wr, w1);
                    }
                }
            }
            small_dft<R, C>(v[q], +1);
        }
    }
    if (last) {
        // Ns R = h: j < Ns, output z_{j + r nb} = pixels 2 (j + r nb), 2 (j + r nb) + 1
        const bool al = (reinterpret_cast<uintptr_t>(out) & 15) == 0;
        double2 *o2 = reinterpret_cast<double2 *>(out);
        // pixels are float64 whatever the precision of the passes
#pragma unroll
        for (int q = 0; q < MAXQ; ++q) {
            const int j = tid + q * NT;
            if (store && j < nb) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int i = j + r * nb;
                    if (al) {
                        o2[i] = todbl(v[q][r]);
                    } else {
                        out[2 * i] = (double)v[q][r].x;
                        out[2 * i + 1] = (double)v[q][r].y;
                    }
                }
            }
        }
    } else {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < MAXQ; ++q) {
            const int j = tid + q * NT;
            if (j < nb) {
                const int jq = (Ns == 1) ? j : (int)__umulhi((unsigned)j, magic);
                const int base = jq * Ns * R + (j - jq * Ns);
#pragma unroll
                for (int r = 0; r < R; ++r) buf[PadIdx::at(base + r * Ns)] = v[q][r];
            }
        }
        __syncthreads();
    }
}

// Fold of a fast-path ring (modes m = 0..mmax <= kFastMaxModes - 1, n even).
// Every thread loads its modes m = tid + q NT at once, multiplies them by
// e^{i m phi0} and stores them at buf[PadIdx(m)]; then bin k sums its
// aliases m = k + j n and conj of m = j n - k in a fixed order (j ascending,
// direct before mirrored), in place: below index n/2 + 1 the buffer entry m
// is read only by bin m, whose own thread then overwrites it with F_m.  Rings
// with fewer bins than threads split each bin's aliases over G = NT / bins
// threads and add the G partial sums in a fixed order.  Ends with a barrier.
template <int NT, typename DT>
struct FastModes {
    static constexpr int Q = (kFastMaxModes + NT - 1) / NT;
    DT v[Q];   // as stored (complex64 or complex128), widened at use
};

// Loads of the fold: modes m = tid + q NT of one ring, all at once; they are on
// their way during the passes of the ring before.  paced: each waits for the
// one before it.  The loads of all workgroups then move through the m rows of
// a caller's [m][ring] Delta together, so that the DRAM rows they open serve
// the neighbouring rings too; all at once they reach a Delta beyond the last
// cache as a burst over thousands of rows (delta2map of one l_max 4096 map: 775
// us, paced 736; l_max 2048, whose Delta the cache holds, 217 and 224).
template <int NT, bool PACED = false, typename DT>
__device__ __attribute__((always_inline)) inline void load_fast(FastModes<NT, DT> &raw,
                                                                const DT *__restrict__ drow,
                                                                long long dstride,
                                                                const int *__restrict__ minv,
                                                                int mcontig, int mmax,
                                                                bool paced = false)
{
    constexpr int QM = FastModes<NT, DT>::Q;
    auto pace = [&] {
        // s_waitcnt vmcnt(0) expcnt(7) lgkmcnt(15)
        if (PACED && paced) __builtin_amdgcn_s_waitcnt(0x0F70);
    };
    // an opaque thread index keeps the per-q addresses from being hoisted
    // out of the persistent kernels' ring loop (where they would stay live)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    if (mcontig) {
#pragma unroll
        for (int q = 0; q < QM; ++q) {
            const int m = tid + q * NT;
            raw.v[q] = DT{};
            // uniform: nothing for the rounds of modes that are dead on the ring
            if (q * NT <= mmax && m <= mmax) raw.v[q] = drow[(long long)m * dstride];
            if (q + 1 < QM) pace();
        }
    } else {
        // every position lookup first, then the loads
        int pos[QM];
#pragma unroll
        for (int q = 0; q < QM; ++q) {
            const int m = tid + q * NT;
            pos[q] = (m <= mmax) ? minv[m] : -1;
        }
#pragma unroll
        for (int q = 0; q < QM; ++q) {
            raw.v[q] = (pos[q] >= 0) ? drow[(long long)pos[q] * dstride] : DT{};
            if (q + 1 < QM) pace();
        }
    }
}

template <int NT, typename C>
__device__ __attribute__((always_inline)) inline void fold_bins(C *buf, const RingDesc &d, int mmax);

template <int NT, typename C, typename DT>
__device__ __attribute__((always_inline)) inline void fold_fast(C *buf, const RingDesc &d,
                                                                const FastModes<NT, DT> &raw,
                                                                int mmax)
{
    constexpr int QM = FastModes<NT, DT>::Q;
    const int tid = threadIdx.x;
    double2 ph, step;   // e^{i tid phi0}, e^{i NT phi0}
    {
        double sn, cs;
        sincos((double)tid * d.phi0, &sn, &cs);
        ph = make_double2(cs, sn);
        sincos((double)NT * d.phi0, &sn, &cs);
        step = make_double2(cs, sn);
    }
#pragma unroll
    for (int q = 0; q < QM; ++q) {
        const int m = tid + q * NT;
        if (q * NT > mmax) continue;
        if (m <= mmax) {
            double2 v = widen(raw.v[q]);
            if (m == 0) v.y = 0.0;
            buf[PadIdx::at(m)] = cvt<C>(cmul(ph, v));
        }
        ph = cmul(ph, step);
    }
    __syncthreads();
    fold_bins<NT, C>(buf, d, mmax);
}

// The bins of a fast-path ring from its phased modes, in place (see
// fold_fast).  Ends with a barrier.
template <int NT, typename C>
__device__ __attribute__((always_inline)) inline void fold_bins(C *buf, const RingDesc &d, int mmax)
{
    const int tid = threadIdx.x;
    const int n = d.n;
    const int h = n / 2;
    const int B = h + 1;
    if (n > mmax) {
        // at most one direct mode (m = k) and one mirrored mode (m = n - k)
        for (int k = tid; k <= h; k += NT) {
            double2 F = (k <= mmax) ? todbl(buf[PadIdx::at(k)]) : make_double2(0.0, 0.0);
            if (k >= 1 && n - k <= mmax) F = cadd(F, conjd(todbl(buf[PadIdx::at(n - k)])));
            buf[PadIdx::at(k)] = cvt<C>(F);
        }
    } else if (B >= NT) {
        for (int k = tid; k <= h; k += NT) {
            const int jmax = (mmax + k) / n;
            double sr = 0.0, si = 0.0;
            for (int j = 0; j <= jmax; ++j) {
                if (k + j * n <= mmax) {
                    const double2 v = todbl(buf[PadIdx::at(k + j * n)]);
                    sr += v.x; si += v.y;
                }
                if (j >= 1) {
                    const double2 v = todbl(buf[PadIdx::at(j * n - k)]);
                    sr += v.x; si -= v.y;
                }
            }
            buf[PadIdx::at(k)] = cplx<C>(sr, si);
        }
    } else {
        const int G = NT / B;
        const int kk = tid % B, g = tid / B;
        double sr = 0.0, si = 0.0;
        if (g < G) {
            const int jmax = (mmax + kk) / n;
            for (int j = g; j <= jmax; j += G) {
                if (kk + j * n <= mmax) {
                    const double2 v = todbl(buf[PadIdx::at(kk + j * n)]);
                    sr += v.x; si += v.y;
                }
                if (j >= 1) {
                    const double2 v = todbl(buf[PadIdx::at(j * n - kk)]);
                    sr += v.x; si -= v.y;
                }
            }
        }
        __syncthreads();
        if (g < G) buf[PadIdx::at(g * B + kk)] = cplx<C>(sr, si);
        __syncthreads();
        if (tid < B) {
            // column tid of the partials; entry 0 of it is this thread's own
            double tr = 0.0, ti = 0.0;
            for (int q = 0; q < G; ++q) {
                const double2 v = todbl(buf[PadIdx::at(q * B + tid)]);
                tr += v.x; ti += v.y;
            }
            buf[PadIdx::at(tid)] = cplx<C>(tr, ti);
        }
    }
    __syncthreads();
}

template <int NT, typename C>
__device__ __attribute__((always_inline)) inline void fft_fast(C *buf, const C *T,
                                                               const RingDesc &d,
                                                               double *__restrict__ out, int tid,
                                                               bool store);

// Synthesis of one fast-path ring: buf = padded spectrum buffer, T = LDS
// twiddle table, out = the ring's first pixel.
template <int NT, typename C, typename DT>
__device__ __attribute__((always_inline)) inline void synth_fast(C *buf, C *T,
                                                                 const RingDesc &d,
                                                                 const double2 *__restrict__ pool,
                                                                 const DT *__restrict__ drow,
                                                                 long long dstride,
                                                                 const int *__restrict__ minv,
                                                                 int mcontig, int mmax,
                                                                 double *__restrict__ out)
{
    load_tw<NT>(T, pool + d.tw, d.n);
    FastModes<NT, DT> raw;
    load_fast<NT>(raw, drow, dstride, minv, mcontig, mmax);
    fold_fast<NT>(buf, d, raw, mmax);
    fft_fast<NT, C>(buf, T, d, out, threadIdx.x, true);
}

// DFT with positive sign of the h <= kDirectMax points buf[0..h - 1], in
// place, by direct sums: four threads per output take every fourth term, and
// their sums are added in a fixed order.  T: the 2h-th roots.  The buffer
// holds at least NT entries.  Ends with a barrier.
template <int NT>
__device__ __attribute__((noinline)) void direct_dft(double2 *buf, const double2 *T, int h)
{
    const int tid = threadIdx.x, j = tid % kDirectMax, g = tid / kDirectMax;
    double2 acc = make_double2(0.0, 0.0);
    if (j < h && g < 4) {
        int t = (j * g) % h;
        const int step = (4 * j) % h;
        for (int k = g; k < h; k += 4) {
            acc = cadd(acc, cmul(buf[PadIdx::at(k)], tw_at(T, 2 * t)));
            t += step;
            t = t >= h ? t - h : t;
        }
    }
    __syncthreads();
    if (g < 4) buf[PadIdx::at(tid)] = acc;
    __syncthreads();
    if (tid < h) {
        double2 z = acc;
        for (int q = 1; q < 4; ++q) z = cadd(z, buf[PadIdx::at(q * kDirectMax + tid)]);
        buf[PadIdx::at(tid)] = z;
    }
    __syncthreads();
}

// The Stockham passes of a fast-path ring (after the fold) and the pixel
// stores of the last one.
template <int NT, typename C>
__device__ __attribute__((always_inline)) inline void fft_fast(C *buf, const C *T,
                                                               const RingDesc &d,
                                                               double *__restrict__ out, int tid,
                                                               bool store)
{
    const int h = d.n / 2;
    // no radix list: the direct path, of complex128 rings only (the plan), whose
    // NT threads are the whole workgroup
    if constexpr (sizeof(C) == sizeof(double2)) {
        if (d.rads == 0) {
            C z;
            if (tid < h) {
                const C Fk = buf[PadIdx::at(tid)], Fk2 = buf[PadIdx::at(h - tid)];
                const C e1 = cadd(Fk, conjd(Fk2)), o1 = csub(Fk, conjd(Fk2));
                z = cadd(e1, muli(cmul(tw_at(T, tid), o1), +1));
            }
            __syncthreads();
            if (tid < h) buf[PadIdx::at(tid)] = z;
            __syncthreads();
            direct_dft<NT>(buf, T, h);
            if (tid < h && store) {
                z = buf[PadIdx::at(tid)];
                out[2 * tid] = z.x;
                out[2 * tid + 1] = z.y;
            }
            return;
        }
    }
    int Ns = 1;
    for (int p = 0; p < d.np; ++p) {
        const int R = (int)((d.rads >> (5 * p)) & 31);
        const bool first = p == 0, last = p == d.np - 1;
        switch (R) {
        case 16: fast_pass<16, NT, C>(buf, T, h, Ns, first, last, out, tid, store); break;
        case 8: fast_pass<8, NT, C>(buf, T, h, Ns, first, last, out, tid, store); break;
        case 4: fast_pass<4, NT, C>(buf, T, h, Ns, first, last, out, tid, store); break;
        case 2: fast_pass<2, NT, C>(buf, T, h, Ns, first, last, out, tid, store); break;
        case 7: fast_pass<7, NT, C>(buf, T, h, Ns, first, last, out, tid, store); break;
        case 5: fast_pass<5, NT, C>(buf, T, h, Ns, first, last, out, tid, store); break;
        default: fast_pass<3, NT, C>(buf, T, h, Ns, first, last, out, tid, store); break;
        }
        Ns *= R;
    }
}

// ---------------------------------------------------------------------------
// Fast path, two maps per workgroup (mixed forms, complex64 Delta): maps 2p
// and 2p + 1 of a ring are adjacent in Delta, so one 16-byte load per mode
// brings both; all 512 threads load and fold, then each half of them runs the
// Stockham passes of one map's padded LDS buffer, with common barriers.
// `two` is false for the last map of an odd map count (its partner's loads
// read zeros and its stores are skipped).
constexpr int kFast2Threads = 2 * kFastThreads;

template <int NT>
struct FastModes2 {
    static constexpr int Q = FastModes<NT, float2>::Q;
    float4 v[Q];   // (map 2p, map 2p + 1) of mode tid + q NT
};

template <int NT>
__device__ __attribute__((always_inline)) inline void load_fast2(
    FastModes2<NT> &raw, const float2 *__restrict__ drow, long long dstride,
    const int *__restrict__ minv, int mcontig, int mmax, bool aligned, bool two)
{
    constexpr int QM = FastModes2<NT>::Q;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    if (mcontig && aligned) {
#pragma unroll
        for (int q = 0; q < QM; ++q) {
            const int m = tid + q * NT;
            raw.v[q] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (q * NT <= mmax && m <= mmax)
                raw.v[q] = *reinterpret_cast<const float4 *>(drow + (long long)m * dstride);
        }
        return;
    }
    int pos[QM];
#pragma unroll
    for (int q = 0; q < QM; ++q) {
        const int m = tid + q * NT;
        pos[q] = (m > mmax) ? -1 : (mcontig ? m : minv[m]);
    }
#pragma unroll
    for (int q = 0; q < QM; ++q) {
        float2 e0 = make_float2(0.f, 0.f), e1 = e0;
        if (pos[q] >= 0) {
            const float2 *e = drow + (long long)pos[q] * dstride;
            e0 = e[0];
            if (two) e1 = e[1];
        }
        raw.v[q] = make_float4(e0.x, e0.y, e1.x, e1.y);
    }
}

// fold_fast of 256 threads for both maps, on 512: the same phases and the same
// order of additions per map, so that the outputs do not depend on how many
// threads share a ring.  A thread's modes are every second one of those that
// thread tid % 256 would take alone, and its phases the same powers of
// e^{i 256 phi0}, one product at a time.
template <int NT>
__device__ __attribute__((always_inline)) inline void fold_fast2(float2 *X0, float2 *X1,
                                                                 const RingDesc &d,
                                                                 const FastModes2<NT> &raw,
                                                                 int mmax)
{
    constexpr int QM = FastModes2<NT>::Q;
    static_assert(NT == 2 * kFastThreads, "two phases of a 256-thread fold per round");
    const int tid = threadIdx.x;
    double2 ph, step;   // e^{i m phi0} of this thread's mode, e^{i 256 phi0}
    {
        double sn, cs;
        sincos((double)(tid % kFastThreads) * d.phi0, &sn, &cs);
        ph = make_double2(cs, sn);
        sincos((double)kFastThreads * d.phi0, &sn, &cs);
        step = make_double2(cs, sn);
    }
    if (tid >= kFastThreads) ph = cmul(ph, step);
#pragma unroll
    for (int q = 0; q < QM; ++q) {
        const int m = tid + q * NT;
        if (q * NT > mmax) continue;
        if (m <= mmax) {
            const float4 r = raw.v[q];
            double2 v0 = make_double2((double)r.x, (double)r.y);
            double2 v1 = make_double2((double)r.z, (double)r.w);
            if (m == 0) { v0.y = 0.0; v1.y = 0.0; }
            X0[PadIdx::at(m)] = cvt<float2>(cmul(ph, v0));
            X1[PadIdx::at(m)] = cvt<float2>(cmul(ph, v1));
        }
        ph = cmul(cmul(ph, step), step);
    }
    __syncthreads();
    const int n = d.n;
    const int h = n / 2;
    const int B = h + 1;
    if (n > mmax) {
        for (int k = tid; k <= h; k += NT) {
            double2 F0 = (k <= mmax) ? todbl(X0[PadIdx::at(k)]) : make_double2(0.0, 0.0);
            double2 F1 = (k <= mmax) ? todbl(X1[PadIdx::at(k)]) : make_double2(0.0, 0.0);
            if (k >= 1 && n - k <= mmax) {
                F0 = cadd(F0, conjd(todbl(X0[PadIdx::at(n - k)])));
                F1 = cadd(F1, conjd(todbl(X1[PadIdx::at(n - k)])));
            }
            X0[PadIdx::at(k)] = cvt<float2>(F0);
            X1[PadIdx::at(k)] = cvt<float2>(F1);
        }
    } else if (B >= kFastThreads) {
        for (int k = tid; k <= h; k += NT) {
            const int jmax = (mmax + k) / n;
            double s0r = 0.0, s0i = 0.0, s1r = 0.0, s1i = 0.0;
            for (int j = 0; j <= jmax; ++j) {
                if (k + j * n <= mmax) {
                    const double2 a = todbl(X0[PadIdx::at(k + j * n)]);
                    const double2 c = todbl(X1[PadIdx::at(k + j * n)]);
                    s0r += a.x; s0i += a.y; s1r += c.x; s1i += c.y;
                }
                if (j >= 1) {
                    const double2 a = todbl(X0[PadIdx::at(j * n - k)]);
                    const double2 c = todbl(X1[PadIdx::at(j * n - k)]);
                    s0r += a.x; s0i -= a.y; s1r += c.x; s1i -= c.y;
                }
            }
            X0[PadIdx::at(k)] = cplx<float2>(s0r, s0i);
            X1[PadIdx::at(k)] = cplx<float2>(s1r, s1i);
        }
    } else {
        // G as in fold_fast, so that a ring rounds alike in both
        const int G = kFastThreads / B;
        const int kk = tid % B, g = tid / B;
        double s0r = 0.0, s0i = 0.0, s1r = 0.0, s1i = 0.0;
        if (g < G) {
            const int jmax = (mmax + kk) / n;
            for (int j = g; j <= jmax; j += G) {
                if (kk + j * n <= mmax) {
                    const double2 a = todbl(X0[PadIdx::at(kk + j * n)]);
                    const double2 c = todbl(X1[PadIdx::at(kk + j * n)]);
                    s0r += a.x; s0i += a.y; s1r += c.x; s1i += c.y;
                }
                if (j >= 1) {
                    const double2 a = todbl(X0[PadIdx::at(j * n - kk)]);
                    const double2 c = todbl(X1[PadIdx::at(j * n - kk)]);
                    s0r += a.x; s0i -= a.y; s1r += c.x; s1i -= c.y;
                }
            }
        }
        __syncthreads();
        if (g < G) {
            X0[PadIdx::at(g * B + kk)] = cplx<float2>(s0r, s0i);
            X1[PadIdx::at(g * B + kk)] = cplx<float2>(s1r, s1i);
        }
        __syncthreads();
        if (tid < B) {
            double t0r = 0.0, t0i = 0.0, t1r = 0.0, t1i = 0.0;
            for (int q = 0; q < G; ++q) {
                const double2 a = todbl(X0[PadIdx::at(q * B + tid)]);
                const double2 c = todbl(X1[PadIdx::at(q * B + tid)]);
                t0r += a.x; t0i += a.y; t1r += c.x; t1i += c.y;
            }
            X0[PadIdx::at(tid)] = cplx<float2>(t0r, t0i);
            X1[PadIdx::at(tid)] = cplx<float2>(t1r, t1i);
        }
    }
    __syncthreads();
}

// Persistent over (ring, map pair) items, ring by ring (groups of 2^gshift
// rings go to the XCDs in turn, ring_group).  LDS: two spectra of lds.fft_entries each, then the
// twiddle table.
__global__ __launch_bounds__(kFast2Threads, 4) void k_ring_synth_fast2(
    const int *__restrict__ ids, int count, int nmaps, const RingDesc *__restrict__ rings,
    const float2 *__restrict__ pool32, const float2 *__restrict__ delta,
    const int *__restrict__ minv, int mcontig, DeltaLayout dl,
    double *__restrict__ map, long long npix, RingLds lds, int gshift)
{
    extern __shared__ double2 lds_raw[];
    float2 *X0 = reinterpret_cast<float2 *>(lds_raw);
    float2 *X1 = X0 + lds.fft_entries;
    float2 *T = X1 + lds.fft_entries;
    const int npairs = (nmaps + 1) / 2;
    const bool aligned = (nmaps % 2) == 0;
    const int per = (int)(gridDim.x / 8);
    const int x = (int)(blockIdx.x % 8), w = (int)(blockIdx.x / 8);
    long long lo, hi;
    xcd_share<true>(count, npairs, x, gshift, lo, hi);
    long long it = lo + w;
    if (it >= hi) return;
    int i, pi;
    xcd_item<true>(it, count, npairs, x, gshift, i, pi);
    int r = ids[i];
    long long b = 2LL * pi;
    bool two = b + 1 < nmaps;
    FastModes2<kFast2Threads> raw;
    const int half = threadIdx.x / kFastThreads, htid = threadIdx.x % kFastThreads;
    float2 *const X = half ? X1 : X0;
    load_fast2<kFast2Threads>(raw, delta + b * dl.map + dl.row(r), dl.mstride(r), minv, mcontig,
                             rings[r].mlive32, aligned, two);
    for (bool first = true;; first = false) {
        const RingDesc d = rings[r];
        const bool mine = two || half == 0;
        double *out = map + (mine ? b + half : b) * npix + d.start;
        if (!first) __syncthreads();   // the previous ring's last pass has read X0, X1, T
        load_tw<kFast2Threads>(T, pool32 + d.tw, d.n);
        fold_fast2<kFast2Threads>(X0, X1, d, raw, d.mlive32);
        const long long nx = it + per;
        if (nx < hi) {
            xcd_item<true>(nx, count, npairs, x, gshift, i, pi);
            r = ids[i];
            b = 2LL * pi;
            two = b + 1 < nmaps;
            load_fast2<kFast2Threads>(raw, delta + b * dl.map + dl.row(r), dl.mstride(r), minv, mcontig,
                                     rings[r].mlive32, aligned, two);
        }
        fft_fast<kFastThreads, float2>(X, T, d, out, htid, mine);
        if (nx >= hi) break;
        it = nx;
    }
}

// The fast path where fewer than four workgroups fit on a CU, or the Delta is a
// caller's.  Persistent: the grid is a multiple of 8 workgroups; the (map, ring) items,
// in the order of ring_item, are split into 8 contiguous ranges, one per XCD
// (workgroups are dealt to the XCDs round-robin), and the workgroups of an
// XCD take its items in turn.  The loads of a workgroup's
// next ring are issued before the Fourier passes of the current one, so that
// their latency is hidden behind the passes.
// This kernel takes complex128 Delta (FP64 plans, or a caller's Delta): its
// passes run in complex128, two workgroups per CU.  The mixed forms'
// complex64 Delta goes to k_ring_synth_fast2 (two maps per workgroup, the
// passes in complex64).
constexpr int kFastBlocks = 2;

__global__ __launch_bounds__(kFastThreads, kFastBlocks) void k_ring_synth_fast(
    const int *__restrict__ ids, int count, int nmaps, const RingDesc *__restrict__ rings,
    const double2 *__restrict__ pool, const double2 *__restrict__ delta,
    const int *__restrict__ minv, int mcontig, int mfull, int paced, DeltaLayout dl,
    double *__restrict__ map, long long npix, RingLds lds)
{
    extern __shared__ double2 buf[];
    double2 *T = buf + lds.fft_entries;
    const int per = (int)(gridDim.x / 8);
    const int x = (int)(blockIdx.x % 8), w = (int)(blockIdx.x / 8);
    long long lo, hi;
    xcd_share<false>(count, nmaps, x, dl.shift, lo, hi);
    long long it = lo + w;
    if (it >= hi) return;
    int i, bi;
    xcd_item<false>(it, count, nmaps, x, dl.shift, i, bi);
    long long b = bi;
    int r = ids[i];
    FastModes<kFastThreads, double2> raw;
    load_fast<kFastThreads, true>(raw, delta + b * dl.map + dl.row(r), dl.mstride(r), minv,
                                  mcontig, ring_mmax(rings[r], mfull), paced != 0);
    for (bool first = true;; first = false) {
        const RingDesc d = rings[r];
        double *out = map + b * npix + d.start;
        if (!first) __syncthreads();   // the previous ring's last pass has read buf and T
        load_tw<kFastThreads>(T, pool + d.tw, d.n);
        fold_fast<kFastThreads>(buf, d, raw, ring_mmax(d, mfull));
        const long long nx = it + per;
        if (nx < hi) {
            xcd_item<false>(nx, count, nmaps, x, dl.shift, i, bi);
            b = bi;
            r = ids[i];
            load_fast<kFastThreads, true>(raw, delta + b * dl.map + dl.row(r), dl.mstride(r), minv,
                                  mcontig, ring_mmax(rings[r], mfull), paced != 0);
        }
        fft_fast<kFastThreads>(buf, T, d, out, threadIdx.x, true);
        if (nx >= hi) break;
        it = nx;
    }
}

__global__ __launch_bounds__(kFastThreads, 2) void k_ring_synth_batch_fast(
    const int2 *__restrict__ items, const BatchMap *__restrict__ maps,
    double *const *__restrict__ outs, const char *__restrict__ ws, RingLds lds)
{
    extern __shared__ double2 buf[];
    const int2 it = items[xcd_logical(blockIdx.x, gridDim.x)];
    const BatchMap &bm = maps[it.x];
    const RingDesc d = bm.rings[it.y];
    const double2 *delta = reinterpret_cast<const double2 *>(ws + bm.delta_off);
    synth_fast<kFastThreads, double2>(buf, buf + lds.fft_entries, d, bm.pool,
                                      delta + bm.dl.row(it.y), bm.dl.mstride(it.y), bm.minv, bm.mcontig, d.mlive,
                                      outs[it.x] + d.start);
}

// ---------------------------------------------------------------------------
// Bluestein fast path of the mixed forms: even rings whose half length
// h = 2 len has a len that is not 7-smooth.  As in split_bluestein, the
// h-point DFT of Z is z_j = E_j + w^j O_j, z_{j+len} = E_j - w^j O_j
// (w = e^{2 pi i / h}), with E, O the len-point DFTs of Z's even- and
// odd-indexed entries, each a Bluestein transform: a cyclic convolution of
// 7-smooth length nb >= 2 len - 1 with the conjugate chirp.  The two
// convolutions run side by side in two padded complex64 LDS buffers X and Y:
// each Stockham pass takes its butterflies in both, so one barrier pair
// serves the two.  The first forward pass forms Z from the folded spectrum
// and multiplies by the chirp, the first inverse pass multiplies by the
// kernel's spectrum bq, and the last inverse pass multiplies by the chirp,
// combines E and O and writes the pixels.  The chirp
// c_k = e^{i pi k^2 / len} = e^{2 pi i (k^2 mod h) / h} is read from the
// ring's n-th roots (n = 2 h) in LDS.
// What the first pass of a direction reads and the last one writes: the folded
// spectrum, the buffers, the buffers times the kernel's spectrum, or a ring's
// pixels (analysis); the buffers, the pixels, or the transform in X (analysis).
enum BlueIn { kBlueInZ, kBlueInBuf, kBlueInBq, kBlueInPix };
enum BlueOut { kBlueOutBuf, kBlueOutPix, kBlueOutZ };

template <typename C>
struct BlueRing {
    int h, len;
    float inv_h;         // 1 / h, rounded
    const C *bq;         // kernel spectrum DFT^-(conj chirp, wrapped) / nb
    double *out;         // first pixel of the ring (synthesis)
    const double *in;    // the same (analysis)
};

template <typename C>
__device__ inline BlueRing<C> blue_ring(const RingDesc &d, const C *pool)
{
    BlueRing<C> br;
    br.h = d.n / 2;
    br.len = br.h / 2;
    br.inv_h = 1.0f / (float)br.h;
    br.bq = pool + d.bq;
    br.out = nullptr;
    br.in = nullptr;
    return br;
}

// k^2 mod h for k < 2^11 and h < 2^13, exactly: k^2 < 2^22 is exact in
// FP32, and the rounded quotient k^2 * (1/h) is within 0.05 of k^2 / h, so
// one correction either way restores the remainder.
__device__ inline int sq_mod(int k, int h, float inv_h)
{
    const int k2 = k * k;
    const int q = (int)((float)k2 * inv_h);
    int r = k2 - q * h;
    r = (r < 0) ? r + h : r;
    return (r >= h) ? r - h : r;
}

// One pass of radix R over both nb-point buffers (input index j + r nb/R,
// output index (j / Ns) Ns R + j % Ns + r Ns); TB holds the nb-th roots, TW the
// n-th roots.
template <typename C, int NT, int R, int sign>
__device__ __attribute__((always_inline)) inline void blue_pass(C *X, C *Y, const C *TW,
                                                                const C *TB, int L, int Ns, int in,
                                                                int outm, const BlueRing<C> &br)
{
    const int nbf = L / R;   // the plan admits nb / R <= NT: one butterfly per thread
    const int tstep0 = L / (Ns * R);
    const unsigned magic = (unsigned)((0x100000000ull + (unsigned)Ns - 1) / (unsigned)Ns);
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int j = tid;
    C a[R], b[R];
    if (j < nbf) {
        if (in == kBlueInZ || in == kBlueInPix) {
            const int h = br.h;
            const bool al = (reinterpret_cast<uintptr_t>(br.in) & 15) == 0;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int k = j + r * nbf;
                if (k < br.len) {
                    const int t0 = 2 * k, t1 = t0 + 1;
                    const C c = tw_at(TW, 2 * sq_mod(k, h, br.inv_h));
                    C z0, z1;
                    if (sizeof(C) == 16 && in == kBlueInPix) {
                        // the DFT of the analysis has negative sign: conjugated
                        // pixels in, conjugated transform out
                        const double *g = br.in + 2 * t0;
                        if (al) {
                            const double2 p0 = reinterpret_cast<const double2 *>(g)[0];
                            const double2 p1 = reinterpret_cast<const double2 *>(g)[1];
                            z0 = cplx<C>(p0.x, -p0.y);
                            z1 = cplx<C>(p1.x, -p1.y);
                        } else {
                            z0 = cplx<C>(g[0], -g[1]);
                            z1 = cplx<C>(g[2], -g[3]);
                        }
                    } else {
                        // Z_t = (F_t + conj F_{h-t}) + i e^{2 pi i t/n} (F_t - conj F_{h-t}),
                        // t = 2k and 2k + 1
                        const C w0 = tw_at(TW, t0), w1 = tw_at(TW, t1);
                        const C F0 = X[PadIdx::at(t0)], G0 = X[PadIdx::at(h - t0)];
                        const C F1 = X[PadIdx::at(t1)], G1 = X[PadIdx::at(h - t1)];
                        z0 = cadd(cadd(F0, conjd(G0)), muli(cmul(w0, csub(F0, conjd(G0))), +1));
                        z1 = cadd(cadd(F1, conjd(G1)), muli(cmul(w1, csub(F1, conjd(G1))), +1));
                    }
                    a[r] = cmul(z0, c);
                    b[r] = cmul(z1, c);
                } else {
                    a[r] = cplx<C>(0.0, 0.0);
                    b[r] = cplx<C>(0.0, 0.0);
                }
            }
        } else if (in == kBlueInBq) {
            // the kernel spectrum's global loads go out before the LDS reads
            C wq[R];
#pragma unroll
            for (int r = 0; r < R; ++r) wq[r] = br.bq[j + r * nbf];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int k = PadIdx::at(j + r * nbf);
                a[r] = cmul(X[k], wq[r]);
                b[r] = cmul(Y[k], wq[r]);
            }
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int k = PadIdx::at(j + r * nbf);
                a[r] = X[k];
                b[r] = Y[k];
            }
        }
        if (Ns > 1) {
            const int jq = (int)__umulhi((unsigned)j, magic);
            const int ts = tstep0 * (j - jq * Ns);
            if (ts != 0) {
                C w1 = tw_at(TB, ts);
                if (sign < 0) w1.y = -w1.y;
                C wr = w1;
#pragma unroll
                for (int r = 1; r < R; ++r) {
                    a[r] = cmul(a[r], wr);
                    b[r] = cmul(b[r], wr);
                    wr = cmul(wr, w1);
                }
            }
        }
        small_dft<R, C>(a, sign);
        small_dft<R, C>(b, sign);
    }
    if (outm == kBlueOutBuf) {
        __syncthreads();
        if (j < nbf) {
            const int jq = (Ns == 1) ? j : (int)__umulhi((unsigned)j, magic);
            const int base = jq * Ns * R + (j - jq * Ns);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int k = PadIdx::at(base + r * Ns);
                X[k] = a[r];
                Y[k] = b[r];
            }
        }
        __syncthreads();
    } else {
        // j < Ns: outputs o = j + r nbf; for o < len, E_o = c_o a, O_o = c_o b
        const int h = br.h, len = br.len;
        if (outm == kBlueOutZ) __syncthreads();
        if (j < nbf) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int o = j + r * nbf;
                if (o < len) {
                    const C c = tw_at(TW, 2 * sq_mod(o, h, br.inv_h));
                    const C w = tw_at(TW, 2 * o);
                    const C E = cmul(a[r], c);
                    const C t = cmul(w, cmul(b[r], c));
                    if (outm == kBlueOutZ) {
                        X[PadIdx::at(o)] = cadd(E, t);
                        X[PadIdx::at(o + len)] = csub(E, t);
                    } else {
                        const double2 z0 = todbl(cadd(E, t)), z1 = todbl(csub(E, t));
                        double *op = br.out;
                        if ((reinterpret_cast<uintptr_t>(op) & 15) == 0) {
                            double2 *o2 = reinterpret_cast<double2 *>(op);
                            o2[o] = z0;
                            o2[o + len] = z1;
                        } else {
                            op[2 * o] = z0.x;
                            op[2 * o + 1] = z0.y;
                            op[2 * (o + len)] = z1.x;
                            op[2 * (o + len) + 1] = z1.y;
                        }
                    }
                }
            }
        }
        if (outm == kBlueOutZ) __syncthreads();
    }
}

// The passes of one direction of a Bluestein fast-path ring's convolutions:
// sign -1 (forward, its first pass reading in0) or +1 (inverse, its last pass
// writing outl).
template <typename C, int NT, int sign>
__device__ __attribute__((always_inline)) inline void blue_dir(C *X, C *Y, const C *TW,
                                                               const C *TB, const RingDesc &d,
                                                               const BlueRing<C> &br, int in0,
                                                               int outl)
{
    const int L = d.nb;
    int Ns = 1;
    for (int p = 0; p < d.np; ++p) {
        const int R = (int)((d.rads >> (5 * p)) & 31);
        const int in = p > 0 ? kBlueInBuf : in0;
        const int outm = p == d.np - 1 ? outl : kBlueOutBuf;
        switch (R) {
        case 8: blue_pass<C, NT, 8, sign>(X, Y, TW, TB, L, Ns, in, outm, br); break;
        case 4: blue_pass<C, NT, 4, sign>(X, Y, TW, TB, L, Ns, in, outm, br); break;
        case 2: blue_pass<C, NT, 2, sign>(X, Y, TW, TB, L, Ns, in, outm, br); break;
        case 7: blue_pass<C, NT, 7, sign>(X, Y, TW, TB, L, Ns, in, outm, br); break;
        case 5: blue_pass<C, NT, 5, sign>(X, Y, TW, TB, L, Ns, in, outm, br); break;
        default: blue_pass<C, NT, 3, sign>(X, Y, TW, TB, L, Ns, in, outm, br); break;
        }
        Ns *= R;
    }
}

template <typename C, int NT>
__device__ __attribute__((always_inline)) inline void blue_conv(C *X, C *Y, const C *TW,
                                                                const C *TB, const RingDesc &d,
                                                                const BlueRing<C> &br, int in0,
                                                                int outl)
{
    blue_dir<C, NT, -1>(X, Y, TW, TB, d, br, in0, kBlueOutBuf);
    blue_dir<C, NT, +1>(X, Y, TW, TB, d, br, kBlueInBq, outl);
}

// Persistent like k_ring_synth_fast; complex64 Delta only.
// Items are (ring, map pair), ring by ring: one 16-byte load per mode brings
// the modes of maps 2p and 2p + 1 and the two maps
// are then folded and transformed one after the other in the same buffers
// (half the load rounds per map: caps of 16 maps at nside 2048 3.73 ->
// 3.33 ms).  The next pair's loads go out after the second map's fold.
__global__ __launch_bounds__(kBlueThreads, 4) void k_ring_synth_blue(
    const int *__restrict__ ids, int count, int nmaps, const RingDesc *__restrict__ rings,
    const float2 *__restrict__ pool32, const float2 *__restrict__ delta,
    const int *__restrict__ minv, int mcontig, DeltaLayout dl,
    double *__restrict__ map, long long npix, RingLds lds, int gshift)
{
    typedef float2 C;
    constexpr int QM = FastModes2<kBlueThreads>::Q;
    extern __shared__ double2 lds_raw[];
    C *X = reinterpret_cast<C *>(lds_raw);
    C *Y = X + lds.fft_entries;
    C *TW = Y + lds.y_entries;
    C *TB = TW + lds.tw_entries;
    const int npairs = (nmaps + 1) / 2;
    const bool aligned = (nmaps % 2) == 0;
    const int per = (int)(gridDim.x / 8);
    const int x = (int)(blockIdx.x % 8), w = (int)(blockIdx.x / 8);
    long long lo, hi;
    xcd_share<true>(count, npairs, x, gshift, lo, hi);
    long long it = lo + w;
    if (it >= hi) return;
    int i, pi;
    xcd_item<true>(it, count, npairs, x, gshift, i, pi);
    int r = ids[i];
    long long b = 2LL * pi;
    bool two = b + 1 < nmaps;
    FastModes2<kBlueThreads> raw;
    load_fast2<kBlueThreads>(raw, delta + b * dl.map + dl.row(r), dl.mstride(r), minv, mcontig,
                             rings[r].mlive32, aligned, two);
    for (bool first = true;; first = false) {
        const RingDesc d = rings[r];
        BlueRing<C> br = blue_ring<C>(d, pool32);
        br.out = map + b * npix + d.start;
        const bool twoB = two;
        if (!first) __syncthreads();   // the previous ring's last pass has read TW
        load_tw<kBlueThreads>(TW, pool32 + d.tw, d.n);
        load_tw<kBlueThreads>(TB, pool32 + d.twb, d.nb);
        FastModes<kBlueThreads, float2> one;
#pragma unroll
        for (int q = 0; q < QM; ++q) one.v[q] = make_float2(raw.v[q].x, raw.v[q].y);
        fold_fast<kBlueThreads>(X, d, one, d.mlive32);
        blue_conv<C, kBlueThreads>(X, Y, TW, TB, d, br, kBlueInZ, kBlueOutPix);
        br.out += npix;
        if (twoB) {
#pragma unroll
            for (int q = 0; q < QM; ++q) one.v[q] = make_float2(raw.v[q].z, raw.v[q].w);
            __syncthreads();   // the first map's last pass has read X and Y
            fold_fast<kBlueThreads>(X, d, one, d.mlive32);
        }
        const long long nx = it + per;
        if (nx < hi) {
            xcd_item<true>(nx, count, npairs, x, gshift, i, pi);
            r = ids[i];
            b = 2LL * pi;
            two = b + 1 < nmaps;
            load_fast2<kBlueThreads>(raw, delta + b * dl.map + dl.row(r), dl.mstride(r), minv, mcontig,
                                     rings[r].mlive32, aligned, two);
        }
        if (twoB) {
            blue_conv<C, kBlueThreads>(X, Y, TW, TB, d, br, kBlueInZ, kBlueOutPix);
        }
        if (nx >= hi) break;
        it = nx;
    }
}

// ---------------------------------------------------------------------------
// The same path in complex128 (FP64 plans), one map of a ring per workgroup.
// Against the size-class kernels it has both convolutions in one set of passes
// and the chirps, the kernel spectrum, the pre-processing and the stores inside
// them: a third of the barriers.
// Bound by the latency of its passes (LDS and barriers).  Rings of one map,
// against the size-class kernels: nside 512, synthesis 47 to 37 us for the
// stage; nside 2048, analysis 740 to 540 us, synthesis 1.1 to 0.58 ms; a batch
// of 64 maps of l_max 256 to 2048, 3.3 to 2.4 ms for the stage.
template <int NT>
__device__ __attribute__((always_inline)) inline void synth_blue64(
    double2 *X, const RingLds &lds, const RingDesc &d, const double2 *__restrict__ pool,
    const double2 *__restrict__ drow, long long dstride, const int *__restrict__ minv, int mcontig,
    double *__restrict__ out)
{
    double2 *Y = X + lds.fft_entries, *TW = Y + lds.y_entries, *TB = TW + lds.tw_entries;
    const int tid = threadIdx.x, mm = d.mlive;
    load_tw<NT>(TW, pool + d.tw, d.n);
    load_tw<NT>(TB, pool + d.twb, d.nb);
    double2 ph, step;   // e^{i m phi0} of this thread's mode, e^{i NT phi0}
    {
        double sn, cs;
        sincos((double)tid * d.phi0, &sn, &cs);
        ph = make_double2(cs, sn);
        sincos((double)NT * d.phi0, &sn, &cs);
        step = make_double2(cs, sn);
    }
    constexpr int U = 4;
    for (int m0 = tid; m0 <= mm; m0 += U * NT) {
        double2 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int m = m0 + u * NT;
            v[u] = m <= mm ? load_mode(drow, dstride, minv, mcontig, m) : make_double2(0.0, 0.0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int m = m0 + u * NT;
            if (m <= mm) {
                if (m == 0) v[u].y = 0.0;
                X[PadIdx::at(m)] = cmul(ph, v[u]);
            }
            ph = cmul(ph, step);
        }
    }
    __syncthreads();
    fold_bins<NT, double2>(X, d, mm);
    BlueRing<double2> br = blue_ring<double2>(d, pool);
    br.out = out;
    blue_conv<double2, NT>(X, Y, TW, TB, d, br, kBlueInZ, kBlueOutPix);
}

template <int NT>
__global__ __launch_bounds__(NT, 4) void k_ring_synth_blue64(
    const int *__restrict__ ids, int count, int nmaps, const RingDesc *__restrict__ rings,
    const double2 *__restrict__ pool, const double2 *__restrict__ delta,
    const int *__restrict__ minv, int mcontig, DeltaLayout dl, double *__restrict__ map,
    long long npix, RingLds lds)
{
    extern __shared__ double2 buf[];
    int i, b;
    ring_item<false>(xcd_logical(blockIdx.x, gridDim.x), count, nmaps, i, b);
    const int r = ids[i];
    const RingDesc d = rings[r];
    synth_blue64<NT>(buf, lds, d, pool, delta + b * dl.map + dl.row(r), dl.mstride(r), minv,
                     mcontig, map + b * npix + d.start);
}

// The rings of the first complex128 Bluestein class (the first bblocks
// workgroups, bitems rounded up to a multiple of 8) and the fast path's in one
// launch, one workgroup per map and ring: at l_max 512 either alone leaves most
// of the CUs idle (one map: 31.5 us in two launches, 23 in this; 8 maps at
// l_max 1024: 365 us one after the other, 263).  Not persistent: the modes of a next
// ring held through the passes take 218 registers and leave two workgroups on a
// CU; this takes 113, and four workgroups hide the loads better.
__global__ __launch_bounds__(kFastThreads, 4) void k_ring_synth_both(
    int bblocks, const int *__restrict__ bids, int bcount, RingLds blds,
    const int *__restrict__ fids, int fcount, RingLds flds, int nmaps,
    const RingDesc *__restrict__ rings, const double2 *__restrict__ pool,
    const double2 *__restrict__ delta, const int *__restrict__ minv, int mcontig, DeltaLayout dl,
    double *__restrict__ map, long long npix)
{
    extern __shared__ double2 buf[];
    const int block = (int)blockIdx.x;
    int i, b;
    if (block < bblocks) {
        if (block >= bcount * nmaps) return;
        ring_item<false>(xcd_logical(block, bcount * nmaps), bcount, nmaps, i, b);
        const int r = bids[i];
        const RingDesc d = rings[r];
        synth_blue64<kFastThreads>(buf, blds, d, pool, delta + b * dl.map + dl.row(r),
                                   dl.mstride(r), minv, mcontig, map + b * npix + d.start);
        return;
    }
    ring_item<false>(xcd_logical(block - bblocks, fcount * nmaps), fcount, nmaps, i, b);
    const int r = fids[i];
    const RingDesc d = rings[r];
    synth_fast<kFastThreads, double2>(buf, buf + flds.fft_entries, d, pool,
                                      delta + b * dl.map + dl.row(r), dl.mstride(r), minv,
                                      mcontig, d.mlive, map + b * npix + d.start);
}

template <int NT>
__global__ __launch_bounds__(NT, 4) void k_ring_synth_batch_blue64(
    const int2 *__restrict__ items, const BatchMap *__restrict__ maps,
    double *const *__restrict__ outs, const char *__restrict__ ws, RingLds lds)
{
    extern __shared__ double2 buf[];
    const int2 it = items[xcd_logical(blockIdx.x, gridDim.x)];
    const BatchMap &bm = maps[it.x];
    const RingDesc d = bm.rings[it.y];
    const double2 *delta = reinterpret_cast<const double2 *>(ws + bm.delta_off);
    synth_blue64<NT>(buf, lds, d, bm.pool, delta + bm.dl.row(it.y), bm.dl.mstride(it.y), bm.minv,
                     bm.mcontig, outs[it.x] + d.start);
}

template <int NT, int MAXN, typename DT>
__global__ __launch_bounds__(NT, 4) void k_ring_synth(
    const int *__restrict__ ids, int count, int nmaps, const RingDesc *__restrict__ rings,
    const double2 *__restrict__ pool, const DT *__restrict__ delta,
    const int *__restrict__ minv, int mcontig, int mfull, DeltaLayout dl,
    double *__restrict__ map, long long npix, RingLds lds)
{
    extern __shared__ double2 buf[];
    int i, bi;
    ring_item<RingMajor<DT>::value>(xcd_logical(blockIdx.x, gridDim.x), count, nmaps, i, bi);
    const int r = ids[i];
    const long long b = bi;
    const RingDesc d = rings[r];
    double2 *tw = buf + lds.fft_entries;
    const RingTables rt = {tw, tw + lds.tw_entries};
    synth_ring<NT, MAXN, false, false>(buf, rt, d,
                               pool, delta + b * dl.map + dl.row(r), dl.mstride(r), minv,
                               mcontig, ring_mmax<DT>(d, mfull), map + b * npix + d.start);
}

// Batched synthesis: work item (map, ring) of a batch of plans.
template <int NT, int MAXN>
__global__ __launch_bounds__(NT, 4) void k_ring_synth_batch(
    const int2 *__restrict__ items, const BatchMap *__restrict__ maps,
    double *const *__restrict__ outs, const char *__restrict__ ws, RingLds lds)
{
    extern __shared__ double2 buf[];
    const int2 it = items[xcd_logical(blockIdx.x, gridDim.x)];
    const BatchMap &bm = maps[it.x];
    const RingDesc d = bm.crings[it.y];
    const double2 *delta = reinterpret_cast<const double2 *>(ws + bm.delta_off);
    double2 *tw = buf + lds.fft_entries;
    const RingTables rt = {tw, tw + lds.tw_entries};
    synth_ring<NT, MAXN, false, true>(buf, rt, d,
                                bm.pool, delta + bm.dl.row(it.y), bm.dl.mstride(it.y), bm.minv,
                                bm.mcontig,
                                d.mlive, outs[it.x] + d.start);
}

// Analysis (adjoint of the synthesis): G_k by a real DFT, then
// Dt_m = c_m e^{-i m phi0} G_{m mod n} with c_0 = 1 and c_m = cfac for m > 0
// (cfac = 2: the adjoint; cfac = 1: the quadrature analysis), times the
// ring's pixel weight rw[r] when rw is given.
template <int NT, int MAXN>
__global__ __launch_bounds__(NT, 4) void k_ring_anal(
    const int *__restrict__ ids, const RingDesc *__restrict__ rings,
    const double2 *__restrict__ pool, const double *__restrict__ map, long long npix,
    const int *__restrict__ mval, int mcontig, int nm, DeltaLayout dl, double2 *__restrict__ dt,
    int mfull, RingLds lds, const double *__restrict__ rw, double cfac)
{
    extern __shared__ double2 buf[];
    const int r = ids[xcd_logical(blockIdx.x, gridDim.x)];
    const int b = blockIdx.y;
    const RingDesc d = rings[r];
    const RingTables rt = {buf + lds.fft_entries, buf + lds.fft_entries + lds.tw_entries};
    Chirps<NT, MAXN, false> ch;
    ring_tables_load<NT, MAXN, false>(rt, d, pool, ch);
    const double *in = map + (long long)b * npix + d.start;
    const int n = d.n;
    const bool even = (n % 2) == 0;
    const int h = n / 2;
    const int tid = threadIdx.x;
    if (even) {
        if ((reinterpret_cast<uintptr_t>(in) & 15) == 0) {
            const double2 *i2 = reinterpret_cast<const double2 *>(in);
            for (int j = tid; j < h; j += NT) buf[j] = i2[j];
        } else {
            for (int j = tid; j < h; j += NT) buf[j] = make_double2(in[2 * j], in[2 * j + 1]);
        }
        __syncthreads();
        ring_dft<NT, MAXN, false>(buf, d, -1, pool, rt, ch);
        for (int k = tid; k <= h / 2; k += NT) {
            const int k2 = h - k;
            const double2 Zk = buf[k];
            const double2 Zk2 = buf[k2 == h ? 0 : k2];
            // G_k = (Z_k + conj Z_{h-k})/2 - (i/2) e^{-2 pi i k/n} (Z_k - conj Z_{h-k})
            const double2 a1 = cadd(Zk, conjd(Zk2)), b1 = csub(Zk, conjd(Zk2));
            const double2 G1 = csub(a1, muli(cmul(conjd(tw_at(rt.TW, k)), b1), +1));
            const double2 a2 = cadd(Zk2, conjd(Zk)), b2 = csub(Zk2, conjd(Zk));
            const double2 G2 = csub(a2, muli(cmul(conjd(tw_at(rt.TW, k2)), b2), +1));
            buf[k] = make_double2(0.5 * G1.x, 0.5 * G1.y);
            if (k2 != k) buf[k2] = make_double2(0.5 * G2.x, 0.5 * G2.y);
        }
        __syncthreads();
    } else {
        for (int j = tid; j < n; j += NT) buf[j] = make_double2(in[j], 0.0);
        __syncthreads();
        ring_dft<NT, MAXN, false>(buf, d, -1, pool, rt, ch);
    }
    const int kmax = even ? h : n - 1;
    double2 *orow = dt + b * dl.map + dl.row(r);
    const long long om = dl.mstride(r);
    const int mm = ring_mmax(d, mfull);
    double2 step, ph;   // e^{-i NT phi0}, e^{-i m phi0} for this thread's mode
    {
        double sn, cs;
        sincos((double)NT * d.phi0, &sn, &cs);
        step = make_double2(cs, -sn);
    }
    bool first = true;
    const double w = rw ? rw[r] : 1.0;
    for (int i = tid; i < nm; i += NT) {
        const int m = mval[i];
        if (m > mm) break;   // dead on the ring from here on
        const int kk = m % n;
        const double2 G = (kk <= kmax) ? buf[kk] : conjd(buf[n - kk]);
        if (first || !mcontig) {
            double sn, cs;
            sincos((double)m * d.phi0, &sn, &cs);
            ph = make_double2(cs, -sn);
            first = false;
        } else {
            ph = cmul(ph, step);
        }
        double2 v;
        if (m == 0) {
            v = make_double2(G.x, 0.0);
        } else {
            v = cmul(G, ph);
            v.x *= cfac; v.y *= cfac;
        }
        if (rw) { v.x *= w; v.y *= w; }
        orow[i * om] = v;
    }
}

// ---------------------------------------------------------------------------
// Fast path of the analysis: the same rings as the synthesis' (7-smooth half
// length, or a short one by a direct DFT), the same register passes on the
// padded buffer.  The DFT has negative sign: the pixels enter conjugated (as
// z_j = g_2j - i g_{2j+1}) and the passes' results are conjugated where they
// are read.  The first pass takes the pixels straight from the map; G_k of a
// mode is formed from Z_k and Z_{h-k} when the mode is written.
template <int R>
__device__ __attribute__((always_inline)) inline void anal_pass(double2 *buf, const double2 *T,
                                                                int h, int Ns, bool first,
                                                                const double *__restrict__ in)
{
    typedef double2 C;
    constexpr int NT = kFastThreads;
    constexpr int MAXQ = fast_maxq(R);
    const int nb = h / R;
    const int tstep0 = (h / (Ns * R)) * 2;
    const unsigned magic = (unsigned)((0x100000000ull + (unsigned)Ns - 1) / (unsigned)Ns);
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    C v[MAXQ][R];
    const bool al = (reinterpret_cast<uintptr_t>(in) & 15) == 0;
#pragma unroll
    for (int q = 0; q < MAXQ; ++q) {
        const int j = tid + q * NT;
        if (j < nb) {
            if (first) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int i = j + r * nb;
                    v[q][r] = conjd(al ? reinterpret_cast<const C *>(in)[i]
                                       : make_double2(in[2 * i], in[2 * i + 1]));
                }
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r) v[q][r] = buf[PadIdx::at(j + r * nb)];
                const int jq = (int)__umulhi((unsigned)j, magic);
                const int ts = tstep0 * (j - jq * Ns);
                if (ts != 0) {
                    const C w1 = tw_at(T, ts);
                    C wr = w1;
#pragma unroll
                    for (int r = 1; r < R; ++r) {
                        v[q][r] = cmul(v[q][r], wr);
                        wr = cmul(wr, w1);
                    }
                }
            }
            small_dft<R, C>(v[q], +1);
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < MAXQ; ++q) {
        const int j = tid + q * NT;
        if (j < nb) {
            const int jq = first ? j : (int)__umulhi((unsigned)j, magic);
            const int base = jq * Ns * R + (j - jq * Ns);
#pragma unroll
            for (int r = 0; r < R; ++r) buf[PadIdx::at(base + r * Ns)] = v[q][r];
        }
    }
    __syncthreads();
}

// The modes of a ring from conj Z in the padded buffer: Dt_m = c_m e^{-i m phi0}
// G_{m mod n}, times the pixel weight w when `weighted`.  T: the n-th roots.
template <int NT>
__device__ __attribute__((always_inline)) inline void anal_modes(
    const double2 *buf, const double2 *T, const RingDesc &d, const int *__restrict__ mval,
    int mcontig, int nm, int mm, double2 *__restrict__ orow, long long om, double w, bool weighted,
    double cfac)
{
    const int tid = threadIdx.x, n = d.n, h = n / 2;
    double2 step, ph;   // e^{-i NT phi0}, e^{-i m phi0} for this thread's mode
    {
        double sn, cs;
        sincos((double)NT * d.phi0, &sn, &cs);
        step = make_double2(cs, -sn);
    }
    bool first = true;
    for (int i = tid; i < nm; i += NT) {
        const int m = mval[i];
        if (m > mm) break;   // dead on the ring from here on
        if (first || !mcontig) {
            double sn, cs;
            sincos((double)m * d.phi0, &sn, &cs);
            ph = make_double2(cs, -sn);
            first = false;
        } else {
            ph = cmul(ph, step);
        }
        // G_k = (Z_k + conj Z_{h-k})/2 - (i/2) e^{-2 pi i k/n} (Z_k - conj Z_{h-k})
        // (the buffer holds conj Z), and G_{n-k} = conj G_k
        const int kk = m % n, k = kk <= h ? kk : n - kk;
        const double2 Zk = conjd(buf[PadIdx::at(k == h ? 0 : k)]);
        const double2 Zc = buf[PadIdx::at(k == 0 ? 0 : h - k)];
        const double2 a = cadd(Zk, Zc), o = csub(Zk, Zc);
        double2 G = csub(a, muli(cmul(conjd(tw_at(T, k)), o), +1));
        G.x *= 0.5;
        G.y *= kk <= h ? 0.5 : -0.5;
        double2 v;
        if (m == 0) {
            v = make_double2(G.x, 0.0);
        } else {
            v = cmul(G, ph);
            v.x *= cfac; v.y *= cfac;
        }
        if (weighted) { v.x *= w; v.y *= w; }
        orow[i * om] = v;
    }
}

// Ring r of map b.
__device__ __attribute__((always_inline)) inline void anal_fast(
    double2 *buf, int r, int b, const RingDesc *__restrict__ rings,
    const double2 *__restrict__ pool, const double *__restrict__ map, long long npix,
    const int *__restrict__ mval, int mcontig, int nm, const DeltaLayout &dl,
    double2 *__restrict__ dt, int mfull, const RingLds &lds, const double *__restrict__ rw,
    double cfac)
{
    double2 *T = buf + lds.fft_entries;
    const RingDesc d = rings[r];
    const int tid = threadIdx.x;
    const double *in = map + (long long)b * npix + d.start;
    const int n = d.n, h = n / 2;
    load_tw<kFastThreads>(T, pool + d.tw, n);
    if (d.rads == 0) {
        if (tid < h) buf[PadIdx::at(tid)] = make_double2(in[2 * tid], -in[2 * tid + 1]);
        __syncthreads();
        direct_dft<kFastThreads>(buf, T, h);
    } else {
        int Ns = 1;
        for (int p = 0; p < d.np; ++p) {
            const int R = (int)((d.rads >> (5 * p)) & 31);
            switch (R) {
            case 16: anal_pass<16>(buf, T, h, Ns, p == 0, in); break;
            case 8: anal_pass<8>(buf, T, h, Ns, p == 0, in); break;
            case 4: anal_pass<4>(buf, T, h, Ns, p == 0, in); break;
            case 2: anal_pass<2>(buf, T, h, Ns, p == 0, in); break;
            case 7: anal_pass<7>(buf, T, h, Ns, p == 0, in); break;
            case 5: anal_pass<5>(buf, T, h, Ns, p == 0, in); break;
            default: anal_pass<3>(buf, T, h, Ns, p == 0, in); break;
            }
            Ns *= R;
        }
    }
    anal_modes<kFastThreads>(buf, T, d, mval, mcontig, nm, ring_mmax(d, mfull),
                             dt + b * dl.map + dl.row(r), dl.mstride(r), rw ? rw[r] : 1.0, rw != nullptr,
                             cfac);
}

__global__ __launch_bounds__(kFastThreads, 2) void k_ring_anal_fast(
    const int *__restrict__ ids, const RingDesc *__restrict__ rings,
    const double2 *__restrict__ pool, const double *__restrict__ map, long long npix,
    const int *__restrict__ mval, int mcontig, int nm, DeltaLayout dl, double2 *__restrict__ dt,
    int mfull, RingLds lds, const double *__restrict__ rw, double cfac)
{
    extern __shared__ double2 buf[];
    anal_fast(buf, ids[xcd_logical(blockIdx.x, gridDim.x)], blockIdx.y, rings, pool, map, npix,
              mval, mcontig, nm, dl, dt, mfull, lds, rw, cfac);
}

// The Bluestein fast path of the analysis (FP64 plans): ring r of map b.
template <int NT>
__device__ __attribute__((always_inline)) inline void anal_blue64(
    double2 *X, int r, int b, const RingDesc *__restrict__ rings,
    const double2 *__restrict__ pool, const double *__restrict__ map, long long npix,
    const int *__restrict__ mval, int mcontig, int nm, const DeltaLayout &dl,
    double2 *__restrict__ dt, int mfull, const RingLds &lds, const double *__restrict__ rw,
    double cfac)
{
    double2 *Y = X + lds.fft_entries, *TW = Y + lds.y_entries, *TB = TW + lds.tw_entries;
    const RingDesc d = rings[r];
    load_tw<NT>(TW, pool + d.tw, d.n);
    load_tw<NT>(TB, pool + d.twb, d.nb);
    __syncthreads();
    BlueRing<double2> br = blue_ring<double2>(d, pool);
    br.in = map + (long long)b * npix + d.start;
    blue_conv<double2, NT>(X, Y, TW, TB, d, br, kBlueInPix, kBlueOutZ);
    anal_modes<NT>(X, TW, d, mval, mcontig, nm, ring_mmax(d, mfull), dt + b * dl.map + dl.row(r),
                   dl.mstride(r), rw ? rw[r] : 1.0, rw != nullptr, cfac);
}

template <int NT>
__global__ __launch_bounds__(NT, 4) void k_ring_anal_blue64(
    const int *__restrict__ ids, const RingDesc *__restrict__ rings,
    const double2 *__restrict__ pool, const double *__restrict__ map, long long npix,
    const int *__restrict__ mval, int mcontig, int nm, DeltaLayout dl, double2 *__restrict__ dt,
    int mfull, RingLds lds, const double *__restrict__ rw, double cfac)
{
    extern __shared__ double2 buf[];
    anal_blue64<NT>(buf, ids[xcd_logical(blockIdx.x, gridDim.x)], blockIdx.y, rings, pool, map,
                    npix, mval, mcontig, nm, dl, dt, mfull, lds, rw, cfac);
}

// Both in one launch (see k_ring_synth_both): the first bblocks workgroups of a
// map, bcount rounded up to a multiple of 8, take the Bluestein rings.  One map
// at l_max 512: 41 to 21 us; at 2048 (first class only), 93 to 75 us.
__global__ __launch_bounds__(kFastThreads, 4) void k_ring_anal_both(
    const int *__restrict__ fids, int fcount, RingLds flds, const int *__restrict__ bids,
    int bcount, RingLds blds, int bblocks, const RingDesc *__restrict__ rings,
    const double2 *__restrict__ pool, const double *__restrict__ map, long long npix,
    const int *__restrict__ mval, int mcontig, int nm, DeltaLayout dl, double2 *__restrict__ dt,
    int mfull, const double *__restrict__ rw, double cfac)
{
    extern __shared__ double2 buf[];
    const int block = (int)blockIdx.x;
    if (block < bblocks) {
        if (block < bcount)
            anal_blue64<kFastThreads>(buf, bids[xcd_logical(block, bcount)], blockIdx.y, rings,
                                      pool, map, npix, mval, mcontig, nm, dl, dt, mfull, blds, rw,
                                      cfac);
        return;
    }
    anal_fast(buf, fids[xcd_logical(block - bblocks, fcount)], blockIdx.y, rings, pool, map, npix,
              mval, mcontig, nm, dl, dt, mfull, flds, rw, cfac);
}

// Spectrum of the Bluestein kernel b_k = conj(c_k) (wrapped to negative k),
// scaled by 1 / nb, one workgroup per listed ring.
__global__ __launch_bounds__(512) void k_bluestein_prep(
    const RingDesc *__restrict__ rings, const int *__restrict__ ids, double2 *pool)
{
    extern __shared__ double2 buf[];
    const RingDesc d = rings[ids[blockIdx.x]];
    const int len = d.half ? d.clen / 2 : d.clen, nb = d.nb;
    const double2 *chirp = pool + d.tch;
    for (int k = threadIdx.x; k < nb; k += 512) {
        int m = -1;
        if (k < len) m = k;
        else if (k > nb - len) m = nb - k;
        buf[k] = (m >= 0) ? conjd(chirp[m]) : make_double2(0.0, 0.0);
    }
    load_tw<512>(buf + 8192, pool + d.twb, nb);
    __syncthreads();
    fft_lds<512, 8192>(buf, nb, -1, buf + 8192, 1);
    const double inv = 1.0 / (double)nb;
    for (int k = threadIdx.x; k < nb; k += 512)
        pool[d.bq + k] = make_double2(buf[k].x * inv, buf[k].y * inv);
}

// The layout of the ring stage's Delta by its element type.
DeltaLayout delta_layout(const sht_plan_s *p, const float2 *, bool)
{
    return delta_blocked_maps(p->nm, p->nrings, p->nmaps);
}
DeltaLayout delta_layout(const sht_plan_s *p, const double2 *, bool full)
{
    return full ? delta_plain(p->nm, p->nrings) : delta_blocked(p->nm, p->nrings);
}

hipError_t set_lds(const void *fn, size_t bytes)
{
    return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

template <int NT, int MAXN, typename DT>
hipError_t synth_class(const sht_plan_s *p, const RingClass &rc, const DT *delta, double *map,
                       bool full, hipStream_t st)
{
    if (rc.count == 0) return hipSuccess;
    const size_t lds = (size_t)rc.lds.total() * sizeof(double2);
    hipError_t e = set_lds((const void *)k_ring_synth<NT, MAXN, DT>, lds);
    if (e != hipSuccess) return e;
    const long long items = (long long)rc.count * p->nmaps;
    if (items > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((k_ring_synth<NT, MAXN, DT>), dim3((unsigned)items), dim3(NT), lds, st,
                       rc.d_ids, rc.count, p->nmaps, p->d_crings, p->d_pool, delta, p->d_minv,
                       p->mcontig, full ? p->mmax : -1, delta_layout(p, delta, full), map, p->npix,
                       rc.lds);
    return hipGetLastError();
}

template <int NT, int MAXN>
hipError_t anal_class(const sht_plan_s *p, int c, const double *map, double2 *dt, bool full,
                      hipStream_t st, const double *rw, double cfac)
{
    const RingClass &rc = p->cls[c];
    if (rc.count == 0) return hipSuccess;
    const size_t lds =
        (size_t)(rc.lds.fft_entries + rc.lds.tw_entries + rc.lds.tb_entries) * sizeof(double2);
    hipError_t e = set_lds((const void *)k_ring_anal<NT, MAXN>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_ring_anal<NT, MAXN>), dim3((unsigned)rc.count, (unsigned)p->nmaps),
                       dim3(NT), lds, st, rc.d_ids, p->d_crings, p->d_pool, map, p->npix,
                       p->d_mval, p->mcontig, p->nm, delta_layout(p, dt, full), dt,
                       full ? p->mmax : -1, rc.lds, rw, cfac);
    return hipGetLastError();
}

// One launch for the fast path and the first complex128 Bluestein class (if the
// plan has any of it) where four of their workgroups fit on a CU side by side
// (fast-path rings of up to about 4100 pixels); beyond that the longer rings'
// LDS would throttle the shorter ones, and the launches stay apart.
bool rings_together(const sht_plan_s *p)
{
    static_assert(kBlue64Threads[0] == kFastThreads, "one workgroup size for both");
    const RingClass &f = p->scls[kFastClass], &b = p->scls[kBlue64Class];
    return f.count > 0 && f.lds.total() <= kTogetherEntries &&
           (b.count == 0 || b.lds.total() <= kTogetherEntries);
}

size_t together_lds(const sht_plan_s *p)
{
    const RingClass &b = p->scls[kBlue64Class];
    const int f = p->scls[kFastClass].lds.total(), l = b.count > 0 ? b.lds.total() : 0;
    return (size_t)(f > l ? f : l) * sizeof(double2);
}

hipError_t anal_together(const sht_plan_s *p, const double *map, double2 *dt, bool full,
                         hipStream_t st, const double *rw, double cfac)
{
    const RingClass &f = p->scls[kFastClass], &b = p->scls[kBlue64Class];
    const size_t lds = together_lds(p);
    hipError_t e = set_lds((const void *)k_ring_anal_both, lds);
    if (e != hipSuccess) return e;
    const int bblocks = (b.count + 7) / 8 * 8;
    hipLaunchKernelGGL(k_ring_anal_both, dim3((unsigned)(bblocks + f.count), (unsigned)p->nmaps),
                       dim3(kFastThreads), lds, st, f.d_ids, f.count, f.lds, b.d_ids, b.count,
                       b.lds, bblocks, p->d_rings, p->d_pool, map, p->npix, p->d_mval, p->mcontig,
                       p->nm, delta_layout(p, dt, full), dt, full ? p->mmax : -1, rw, cfac);
    return hipGetLastError();
}

// (only an FP64 plan's own Delta is taken together)
hipError_t synth_together(const sht_plan_s *p, const double2 *delta, double *map, hipStream_t st)
{
    const RingClass &f = p->scls[kFastClass], &b = p->scls[kBlue64Class];
    const size_t lds = together_lds(p);
    hipError_t e = set_lds((const void *)k_ring_synth_both, lds);
    if (e != hipSuccess) return e;
    const long long bblocks = ((long long)b.count * p->nmaps + 7) / 8 * 8;
    const long long blocks = bblocks + (long long)f.count * p->nmaps;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(k_ring_synth_both, dim3((unsigned)blocks), dim3(kFastThreads), lds, st,
                       (int)bblocks, b.d_ids, b.count, b.lds, f.d_ids, f.count, f.lds, p->nmaps,
                       p->d_rings, p->d_pool, delta, p->d_minv, p->mcontig,
                       delta_layout(p, delta, false), map, p->npix);
    return hipGetLastError();
}

template <int q>
hipError_t anal_blue64_class(const sht_plan_s *p, const double *map, double2 *dt, bool full,
                             hipStream_t st, const double *rw, double cfac)
{
    const RingClass &rc = p->scls[kBlue64Class + q];
    if (rc.count == 0) return hipSuccess;
    constexpr int NT = kBlue64Threads[q];
    const size_t lds = (size_t)rc.lds.total() * sizeof(double2);
    hipError_t e = set_lds((const void *)k_ring_anal_blue64<NT>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_ring_anal_blue64<NT>, dim3((unsigned)rc.count, (unsigned)p->nmaps),
                       dim3(NT), lds, st, rc.d_ids, p->d_rings, p->d_pool, map, p->npix, p->d_mval,
                       p->mcontig, p->nm, delta_layout(p, dt, full), dt, full ? p->mmax : -1,
                       rc.lds, rw, cfac);
    return hipGetLastError();
}

template <int q>
hipError_t synth_blue64_class(const sht_plan_s *p, const double2 *delta, double *map,
                              hipStream_t st)
{
    const RingClass &rc = p->scls[kBlue64Class + q];
    if (rc.count == 0) return hipSuccess;
    constexpr int NT = kBlue64Threads[q];
    const size_t lds = (size_t)rc.lds.total() * sizeof(double2);
    hipError_t e = set_lds((const void *)k_ring_synth_blue64<NT>, lds);
    if (e != hipSuccess) return e;
    const long long items = (long long)rc.count * p->nmaps;
    if (items > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(k_ring_synth_blue64<NT>, dim3((unsigned)items), dim3(NT), lds, st, rc.d_ids,
                       rc.count, p->nmaps, p->d_rings, p->d_pool, delta, p->d_minv, p->mcontig,
                       delta_layout(p, delta, false), map, p->npix, rc.lds);
    return hipGetLastError();
}

hipError_t anal_fast_class(const sht_plan_s *p, const double *map, double2 *dt, bool full,
                           hipStream_t st, const double *rw, double cfac)
{
    const RingClass &rc = p->scls[kFastClass];
    if (rc.count == 0) return hipSuccess;
    const size_t lds = (size_t)rc.lds.total() * sizeof(double2);
    hipError_t e = set_lds((const void *)k_ring_anal_fast, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_ring_anal_fast, dim3((unsigned)rc.count, (unsigned)p->nmaps),
                       dim3(kFastThreads), lds, st, rc.d_ids, p->d_rings, p->d_pool, map, p->npix,
                       p->d_mval, p->mcontig, p->nm, delta_layout(p, dt, full), dt,
                       full ? p->mmax : -1, rc.lds, rw, cfac);
    return hipGetLastError();
}

}  // namespace

// Size classes (FFT length limit): 0 -> 2048, 1 -> 4096, 2 -> 8192.
static_assert(kClassThreads[0] == 256 && kClassThreads[1] == 512 && kClassThreads[2] == 1024,
              "class thread counts must match the kernel instantiations");
hipError_t synth_fast_class(const sht_plan_s *p, const double2 *delta, double *map, bool full,
                            hipStream_t st)
{
    const RingClass &rc = p->scls[kFastClass];
    if (rc.count == 0) return hipSuccess;
    const size_t lds = (size_t)rc.lds.total() * sizeof(double2);
    hipError_t e = set_lds((const void *)k_ring_synth_fast, lds);
    if (e != hipSuccess) return e;
    // as many workgroups per CU as the LDS of a ring allows (two), a multiple of 8
    const long long items = (long long)rc.count * p->nmaps;
    long long grid = (long long)kFastBlocks * (p->num_cus > 0 ? p->num_cus : 256);
    if (grid > items) grid = items;
    grid = ((grid + 7) / 8) * 8;
    // one map's Delta against the last cache's 256 MB
    const bool past_cache = (long long)p->nm * p->nrings * (long long)sizeof(double2) > (256LL << 20);
    hipLaunchKernelGGL(k_ring_synth_fast, dim3((unsigned)grid), dim3(kFastThreads), lds,
                       st, rc.d_ids, rc.count, p->nmaps, p->d_rings, p->d_pool, delta,
                       p->d_minv, p->mcontig, full ? p->mmax : -1, full && past_cache ? 1 : 0,
                       delta_layout(p, delta, full), map, p->npix, rc.lds);
    return hipGetLastError();
}

// complex64 Delta: two maps per workgroup, two workgroups per CU.
hipError_t synth_fast_class(const sht_plan_s *p, const float2 *delta, double *map, bool full,
                            hipStream_t st)
{
    const RingClass &rc = p->scls[kFastClass];
    if (rc.count == 0) return hipSuccess;
    if (!p->d_pool32) return hipErrorInvalidConfiguration;
    const size_t lds =
        (size_t)(2 * rc.lds.fft_entries + rc.lds.tw_entries) * sizeof(float2);
    hipError_t e = set_lds((const void *)k_ring_synth_fast2, lds);
    if (e != hipSuccess) return e;
    const long long items = (long long)rc.count * ((p->nmaps + 1) / 2);
    long long grid = 2LL * (p->num_cus > 0 ? p->num_cus : 256);
    if (grid > items) grid = items;
    grid = ((grid + 7) / 8) * 8;
    const DeltaLayout dl = delta_layout(p, delta, full);
    hipLaunchKernelGGL(k_ring_synth_fast2, dim3((unsigned)grid), dim3(kFast2Threads), lds, st,
                       rc.d_ids, rc.count, p->nmaps, p->d_rings, p->d_pool32, delta, p->d_minv,
                       p->mcontig, dl, map, p->npix, rc.lds,
                       ring_group(rc.count, (p->nmaps + 1) / 2, grid, dl.shift));
    return hipGetLastError();
}

// The Bluestein fast path (complex64 Delta only): two 512-thread
// workgroups per CU, persistent.
hipError_t synth_blue_class(const sht_plan_s *p, const float2 *delta, double *map, bool full,
                            hipStream_t st)
{
    const RingClass &rc = p->scls[kBlueClass];
    if (rc.count == 0) return hipSuccess;
    if (!p->d_pool32) return hipErrorInvalidConfiguration;
    const size_t lds = (size_t)rc.lds.total() * sizeof(float2);
    hipError_t e = set_lds((const void *)k_ring_synth_blue, lds);
    if (e != hipSuccess) return e;
    const long long items = (long long)rc.count * ((p->nmaps + 1) / 2);
    long long grid = 2LL * (p->num_cus > 0 ? p->num_cus : 256);
    if (grid > items) grid = items;
    grid = ((grid + 7) / 8) * 8;
    const DeltaLayout dl = delta_layout(p, delta, full);
    hipLaunchKernelGGL(k_ring_synth_blue, dim3((unsigned)grid), dim3(kBlueThreads), lds, st,
                       rc.d_ids, rc.count, p->nmaps, p->d_rings, p->d_pool32, delta, p->d_minv,
                       p->mcontig, dl, map, p->npix, rc.lds,
                       ring_group(rc.count, (p->nmaps + 1) / 2, grid, dl.shift));
    return hipGetLastError();
}

// complex128 Delta: an FP64 plan's own goes to the complex128 path; a caller's
// has modes that this path's buffers do not hold (FP64 plans) or that the plan
// never transforms (mixed-form plans): those rings by size class.
hipError_t synth_blue_class(const sht_plan_s *p, const double2 *delta, double *map, bool full,
                            hipStream_t st)
{
    if (!full) {
        hipError_t e = synth_blue64_class<2>(p, delta, map, st);
        if (e == hipSuccess) e = synth_blue64_class<1>(p, delta, map, st);
        if (e == hipSuccess && !rings_together(p)) e = synth_blue64_class<0>(p, delta, map, st);
        return e;
    }
    hipError_t e = synth_class<1024, 8192, double2>(p, p->bcls[2], delta, map, full, st);
    if (e == hipSuccess) e = synth_class<512, 4096, double2>(p, p->bcls[1], delta, map, full, st);
    if (e == hipSuccess) e = synth_class<256, 2048, double2>(p, p->bcls[0], delta, map, full, st);
    return e;
}

// The fast-path kernel (LDS-bound at two or three workgroups per CU), the
// Bluestein fast path and the size-class kernels write disjoint rings.  For
// large plans the fast path runs on the plan's auxiliary stream beside the
// others (forked from and joined back into the caller's stream by events, so
// the call stays ordered on `st` and capturable): their workgroups then
// share the CUs and fill each other's tails (FP64 size classes: 10.6 -> 10.2
// ms for 16 maps at l_max 4096 / nside 2048; with the mixed forms' two fast
// paths: 5.93 -> 5.84 ms).
// Small plans launch everything on `st` (a fork costs microseconds).  The
// mixed forms' two kernels fill the CUs each by itself and only gain from
// larger launches on (FP16x2, 16 maps, transform forked against in turn: nside
// 192 238 and 224 us, 200 288 and 230, 216 334 and 275, 300 416 and 409, 400
// and 500 alike; 600 1095 and 1103).
constexpr long long kForkItems = 4096;
constexpr long long kForkItemsMixed = 32768;

template <typename DT> constexpr bool own_complex128(bool full)
{
    return sizeof(DT) == sizeof(double2) && !full;
}

template <typename DT>
static hipError_t ring_synth_dt(const sht_plan_s *p, const DT *delta, double *map, bool full,
                                hipStream_t st)
{
    const bool both = own_complex128<DT>(full) && rings_together(p);
    long long fast = p->scls[kFastClass].count, rest = 0;
    for (int q = 0; q < kNumSynthClasses; ++q)
        if (q != kFastClass) rest += p->scls[q].count;
    if (both) {
        fast += p->scls[kBlue64Class].count;
        rest -= p->scls[kBlue64Class].count;
    }
    fast *= p->nmaps;
    rest *= p->nmaps;
    const bool fork = p->aux_stream && fast > 0 && rest > 0 &&
                      fast + rest >= (sizeof(DT) == sizeof(float2) ? kForkItemsMixed : kForkItems);
    // the fork and join events belong to the plan: calls from several host
    // threads take turns through the whole sequence
    std::unique_lock<std::mutex> lock(const_cast<sht_plan_s *>(p)->fork_mu, std::defer_lock);
    if (fork) lock.lock();
    hipError_t e = hipSuccess;
    if (fork) {
        e = hipEventRecord(p->ev_fork, st);
        if (e == hipSuccess) e = hipStreamWaitEvent(p->aux_stream, p->ev_fork, 0);
    }
    const hipStream_t fst = fork ? p->aux_stream : st;
    if (e == hipSuccess) {
        if constexpr (sizeof(DT) == sizeof(double2)) {
            e = both ? synth_together(p, delta, map, fst)
                     : synth_fast_class(p, delta, map, full, fst);
        } else {
            e = synth_fast_class(p, delta, map, full, fst);
        }
    }
    if (e == hipSuccess) e = synth_blue_class(p, delta, map, full, st);
    if (e == hipSuccess) e = synth_class<1024, 8192, DT>(p, p->scls[2], delta, map, full, st);
    if (e == hipSuccess) e = synth_class<512, 4096, DT>(p, p->scls[1], delta, map, full, st);
    if (e == hipSuccess) e = synth_class<256, 2048, DT>(p, p->scls[0], delta, map, full, st);
    if (fork) {
        // join even after a failed launch, so that `st` never runs ahead of
        // work already queued on the auxiliary stream
        const hipError_t j = hipEventRecord(p->ev_join, p->aux_stream);
        const hipError_t w = (j == hipSuccess) ? hipStreamWaitEvent(st, p->ev_join, 0) : j;
        if (e == hipSuccess) e = w;
    }
    return e;
}

hipError_t launch_ring_synth(const sht_plan_s *p, const double2 *delta, double *map, bool full,
                             hipStream_t st)
{
    return ring_synth_dt(p, delta, map, full, st);
}

hipError_t launch_ring_synth(const sht_plan_s *p, const float2 *delta, double *map,
                             hipStream_t st)
{
    return ring_synth_dt(p, delta, map, false, st);
}

// Complex64 Delta widened to complex128 (the stage entry point's layout).
__global__ __launch_bounds__(256) void k_narrow(const double2 *__restrict__ s,
                                                float2 *__restrict__ d, long long n)
{
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i < n) d[i] = make_float2((float)s[i].x, (float)s[i].y);
}

hipError_t launch_narrow(const double2 *s, float2 *d, long long n, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const long long nb = (n + 255) / 256;
    if (nb > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(k_narrow, dim3((unsigned)nb), dim3(256), 0, st, s, d, n);
    return hipGetLastError();
}

// complex64 Delta of the mixed forms -> complex128 [map][m][ring] (exact), one
// thread per output entry.
__global__ __launch_bounds__(256) void k_widen_delta(const float2 *__restrict__ s, DeltaLayout dl,
                                                     double2 *__restrict__ d, int nmaps, int nm,
                                                     int nrings)
{
    const long long n = (long long)nmaps * nm * nrings;
    const long long o = (long long)blockIdx.x * 256 + threadIdx.x;
    if (o >= n) return;
    const int r = (int)(o % nrings);
    const long long t = o / nrings;
    const int i = (int)(t % nm);
    const float2 v = s[(t / nm) * dl.map + dl.row(r) + i * dl.mstride(r)];
    d[o] = make_double2((double)v.x, (double)v.y);
}

hipError_t launch_widen_delta(const sht_plan_s *p, const float2 *s, double2 *d, hipStream_t st)
{
    const long long n = (long long)p->nmaps * p->nm * p->nrings;
    if (n <= 0) return hipSuccess;
    const long long nb = (n + 255) / 256;
    if (nb > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(k_widen_delta, dim3((unsigned)nb), dim3(256), 0, st, s,
                       delta_layout(p, s, false), d, p->nmaps, p->nm,
                       p->nrings);
    return hipGetLastError();
}

hipError_t launch_ring_anal(const sht_plan_s *p, const double *map, double2 *dt, bool full,
                            hipStream_t st, const double *rw, double cfac)
{
    const bool both = p->anal_fast && rings_together(p);
    hipError_t e = hipSuccess;
    if (both)
        e = anal_together(p, map, dt, full, st, rw, cfac);
    else if (p->anal_fast)
        e = anal_fast_class(p, map, dt, full, st, rw, cfac);
    if (e == hipSuccess) e = anal_blue64_class<2>(p, map, dt, full, st, rw, cfac);
    if (e == hipSuccess) e = anal_blue64_class<1>(p, map, dt, full, st, rw, cfac);
    if (e == hipSuccess && !both) e = anal_blue64_class<0>(p, map, dt, full, st, rw, cfac);
    if (e == hipSuccess) e = anal_class<1024, 8192>(p, 2, map, dt, full, st, rw, cfac);
    if (e == hipSuccess) e = anal_class<512, 4096>(p, 1, map, dt, full, st, rw, cfac);
    if (e == hipSuccess) e = anal_class<256, 2048>(p, 0, map, dt, full, st, rw, cfac);
    return e;
}

// r = s - r over n doubles (residual of the refined analysis)
__global__ __launch_bounds__(256) void k_residual(const double *__restrict__ s,
                                                  double *__restrict__ r, long long n)
{
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i < n) r[i] = s[i] - r[i];
}

hipError_t launch_residual(const double *s, double *r, long long n, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const long long nb = (n + 255) / 256;
    if (nb > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(k_residual, dim3((unsigned)nb), dim3(256), 0, st, s, r, n);
    return hipGetLastError();
}

template <int NT, int MAXN>
hipError_t synth_batch_class(const BatchClass &bc, const BatchMap *maps, double *const *outs,
                             const void *ws, hipStream_t st)
{
    if (bc.count == 0) return hipSuccess;
    const size_t lds = (size_t)bc.lds.total() * sizeof(double2);
    hipError_t e = set_lds((const void *)k_ring_synth_batch<NT, MAXN>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_ring_synth_batch<NT, MAXN>), dim3((unsigned)bc.count), dim3(NT), lds, st,
                       bc.d_items, maps, outs, (const char *)ws, bc.lds);
    return hipGetLastError();
}

template <int q>
hipError_t synth_batch_blue64(const BatchClass *cls, const BatchMap *maps, double *const *outs,
                              const void *ws, hipStream_t st)
{
    const BatchClass &bc = cls[kBlue64Class + q];
    if (bc.count == 0) return hipSuccess;
    constexpr int NT = kBlue64Threads[q];
    const size_t lds = (size_t)bc.lds.total() * sizeof(double2);
    hipError_t e = set_lds((const void *)k_ring_synth_batch_blue64<NT>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_ring_synth_batch_blue64<NT>, dim3((unsigned)bc.count), dim3(NT), lds, st,
                       bc.d_items, maps, outs, (const char *)ws, bc.lds);
    return hipGetLastError();
}

hipError_t launch_ring_synth_batch(const BatchClass *cls, const BatchMap *maps,
                                   double *const *outs, const void *ws, hipStream_t st)
{
    hipError_t e = hipSuccess;
    const BatchClass &fc = cls[kFastClass];
    if (fc.count > 0) {
        const size_t lds = (size_t)fc.lds.total() * sizeof(double2);
        e = set_lds((const void *)k_ring_synth_batch_fast, lds);
        if (e == hipSuccess) {
            hipLaunchKernelGGL(k_ring_synth_batch_fast, dim3((unsigned)fc.count),
                               dim3(kFastThreads), lds, st, fc.d_items, maps, outs,
                               (const char *)ws, fc.lds);
            e = hipGetLastError();
        }
    }
    if (e == hipSuccess) e = synth_batch_blue64<2>(cls, maps, outs, ws, st);
    if (e == hipSuccess) e = synth_batch_blue64<1>(cls, maps, outs, ws, st);
    if (e == hipSuccess) e = synth_batch_blue64<0>(cls, maps, outs, ws, st);
    if (e == hipSuccess) e = synth_batch_class<1024, 8192>(cls[2], maps, outs, ws, st);
    if (e == hipSuccess) e = synth_batch_class<512, 4096>(cls[1], maps, outs, ws, st);
    if (e == hipSuccess) e = synth_batch_class<256, 2048>(cls[0], maps, outs, ws, st);
    return e;
}

hipError_t launch_bluestein_prep(const sht_plan_s *p, const RingDesc *rings, const int *ring_ids,
                                 int nids, hipStream_t st)
{
    if (nids <= 0) return hipSuccess;
    const size_t lds = (size_t)(8192 + kTwEntries) * sizeof(double2);
    hipError_t e = set_lds((const void *)k_bluestein_prep, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_bluestein_prep, dim3((unsigned)nids), dim3(512), lds, st,
                       rings, ring_ids, p->d_pool);
    return hipGetLastError();
}

}  // namespace sht
