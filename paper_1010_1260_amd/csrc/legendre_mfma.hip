// Mixed-precision batched Legendre stage on the matrix cores (gfx950), FP32
// operands.
//
// For a batch of maps sharing one geometry, Delta_m(theta) of Eq. (DeltaDef)
// is, per m, a matrix product: with ring pairs as columns, l as the inner
// index and (map, Re/Im) as rows,
//     C_E = B_E[rows x K] * Lambda_E[K x pairs]   (l - m even)
//     C_O = B_O[rows x K] * Lambda_O[K x pairs]   (l - m odd)
//     Delta_N = C_E + C_O,  Delta_S = C_E - C_O.
// The recurrence (Eq. assLegRec) stays in FP64 on the vector ALUs, exactly as
// in the FP64 kernel, each pair from its start row on (live.hip); only the true
// values P_lm, rounded to FP32, and the FP32 copy of the prescaled
// coefficients enter the matrix core.
//
// Fragments.  v_mfma_f32_4x4x1_16b multiplies, in each of 16 blocks of four
// lanes, a column of four rows by a row of four pairs.  Lane = ring pair: the
// lane's own P_lm is the second operand as it stands, and its four sums (two
// maps' Re and Im) come out in the lane.  The first operand holds the
// coefficients of 16 rows l of two maps, four lanes each, and the
// instruction's block broadcast picks the row: one register per two maps
// feeds 16 products, and the work goes with the number of maps (a 32x32
// tile always pays for 16).  Every product adds one term, so the sums run in
// the order of l whatever the number of maps.
//
// Work split.  One wave per (64 ring pairs, m-pair, up to 16 maps); the waves
// share nothing.  A block's coefficients (256 bytes per two maps) are asked
// for a block ahead, A_l through scalar registers half a block ahead.
//
// Accumulation.  FP32 accumulation over all l-terms loses up to ~1e-6; the
// matrix core accumulates the 64 same-parity terms of a super-block from zero
// and the block sums are added into a second FP32 accumulator (two-level
// summation).  Emulated error of Delta at l_max = 4096: about 1.2e-7 relative.
//
// Bound: the matrix core (8 cycles per row and two maps) plus the vector work
// (12 cycles per row); FP32 matrix and FP64 vector instructions take turns.
// l_max 1999 / nside 999, 5 maps: 1.14 ms; 2.71 ms on 32x32x2 tiles of 16 maps,
// four waves sharing the coefficients in LDS, every row from l = m on.  The
// whole transform at l_max 1024 / nside 512: one map 521 -> 213 us, 8 maps 819
// -> 596 us, 16 maps 1209 -> 1128 us; l_max 4096, 16 maps 27.3 -> 23.2 ms.
#include <type_traits>

#include "mixed_common.h"

namespace sht {
namespace {

constexpr int kBlk = 16;                    // l-rows per block
constexpr int kSuper = 8;                   // blocks per super-block: 64 terms per parity
constexpr int kSuperRows = kSuper * kBlk;
constexpr int kMaxPairs = 8;                // map pairs of a group (16 maps)

// Packed B of a group of np map pairs, block b of an m: [map pair][lane 64],
// lane i + 4 (r + 8 p) holding row 16 b + 2 r + p (p: parity) of map
// i / 2 of the pair (Re for even i, Im for odd), i.e. a'_lm = c_lm a_lm, zero
// past the m's last row.  One workgroup per kPreBlocks consecutive blocks
// (bm16: the m of each block): the a_lm are read in runs of 16 rows per map
// (each complex value once), and the packed blocks are assembled in LDS and
// written out contiguously.
constexpr int kPreBlocks = 8;

__global__ __launch_bounds__(256) void k_prescale_f32(
    const double2 *__restrict__ alm, const double *__restrict__ cn,
    const long long *__restrict__ moff, const int *__restrict__ mval,
    const long long *__restrict__ boff16, const int *__restrict__ bm16, int lmax,
    long long nalm, long long nblocks, int nmaps, int np, long long m0len,
    float *__restrict__ Bp)
{
    __shared__ __attribute__((aligned(16))) float stage[kPreBlocks * kMaxPairs * 64];
    const long long blk0 = (long long)blockIdx.x * kPreBlocks;
    const int nb = (int)min((long long)kPreBlocks, nblocks - blk0);
    const long long map0 = (long long)blockIdx.y * 2 * np;
    const int tid = threadIdx.x;
    const int rb = tid & 15;                       // row
    for (int w = tid >> 4; w < nb * 2 * np; w += 16) {
        const int b = w / (2 * np), mp = w - b * 2 * np;   // block, map
        const int i = bm16[blk0 + b];
        const int len = lmax - mval[i] + 1;
        const long long row = (blk0 + b - boff16[i]) * kBlk + rb;
        float vr = 0.0f, vi = 0.0f;
        if (row < len && map0 + mp < nmaps) {
            const long long e = moff[i] + row;
            const double2 a = alm[(map0 + mp) * nalm + e];
            const double c = cn[e];
            vr = (float)(a.x * c);
            vi = (float)((e < m0len) ? 0.0 : a.y * c);
        }
        float *s = stage + (b * np + (mp >> 1)) * 64 + 2 * (mp & 1) +
                   4 * ((rb >> 1) + 8 * (rb & 1));
        s[0] = vr;
        s[1] = vi;
    }
    __syncthreads();
    const float4 *s4 = reinterpret_cast<const float4 *>(stage);
    float4 *o4 = reinterpret_cast<float4 *>(
        Bp + ((long long)blockIdx.y * nblocks + blk0) * np * 64);
    for (int w = tid; w < nb * np * 16; w += 256) o4[w] = s4[w];
}

template <int NP>
struct Sums {
    v4f e[NP], o[NP];
};

// Row r (0..7) of both parities of a block: e, o = P_lm of the lane's ring
// pair.  ZERO: the row starts the sums.
template <int NP, int r, bool ZERO>
__device__ __forceinline__ void products(const float (&B)[NP], float e, float o, Sums<NP> &acc)
{
#pragma unroll
    for (int p = 0; p < NP; ++p)
        acc.e[p] = __builtin_amdgcn_mfma_f32_4x4x1f32(B[p], e, ZERO ? v4f{} : acc.e[p], 4, r, 0);
#pragma unroll
    for (int p = 0; p < NP; ++p)
        acc.o[p] =
            __builtin_amdgcn_mfma_f32_4x4x1f32(B[p], o, ZERO ? v4f{} : acc.o[p], 4, 8 + r, 0);
}

template <int NP, int r, bool ZERO>
__device__ __forceinline__ void two_rows(Lane &l, const double *a, const float (&B)[NP],
                                         Sums<NP> &acc)
{
    const double u0 = fma(a[2 * r] * l.x, l.ub, -l.ua);
    const double u1 = fma(a[2 * r + 1] * l.x, u0, -l.ub);
    l.ua = u0;
    l.ub = u1;
    products<NP, r, ZERO>(B, (float)u0, (float)u1, acc);
}

template <int NP>
struct MState {
    int i, nblk, q0;     // blocks of the m, the first one with a live row of the wave
    int hi8;             // the last row at which a pair starts
    const double *Am;    // padded coefficients of the m, per super-block
    const float *Bm;     // its packed blocks, the lane's first value
    Lane l;
    double a[kBlk];
    float B[NP];

    __device__ __forceinline__ void load(float (&b)[NP], int q) const
    {
        const float *s = Bm + (long long)q * (NP * 64);
#pragma unroll
        for (int p = 0; p < NP; ++p) b[p] = s[p * 64];
    }
};

// One block of 16 rows; FIRST: of a super-block.  qn: the block wanted next.
template <int NP, bool FIRST>
__device__ __forceinline__ void block16(MState<NP> &st, const double2 *stash, int q, int qn,
                                        Sums<NP> &acc)
{
    double an[kBlk];
    float Bn[NP];
    scalars_arrived();
    scalar_rows<kBlk>(an, (CDp)st.Am + qn * kBlk);
    __builtin_amdgcn_sched_barrier(0);
    st.load(Bn, qn);
    enter(st.l, stash, q * kBlk, st.hi8);
    two_rows<NP, 0, FIRST>(st.l, st.a, st.B, acc);
    two_rows<NP, 1, false>(st.l, st.a, st.B, acc);
    two_rows<NP, 2, false>(st.l, st.a, st.B, acc);
    two_rows<NP, 3, false>(st.l, st.a, st.B, acc);
    enter(st.l, stash, q * kBlk + 8, st.hi8);
    two_rows<NP, 4, false>(st.l, st.a, st.B, acc);
    two_rows<NP, 5, false>(st.l, st.a, st.B, acc);
    two_rows<NP, 6, false>(st.l, st.a, st.B, acc);
    two_rows<NP, 7, false>(st.l, st.a, st.B, acc);
#pragma unroll
    for (int t = 0; t < kBlk; ++t) st.a[t] = an[t];
#pragma unroll
    for (int p = 0; p < NP; ++p) st.B[p] = Bn[p];
}

// Start of an m: the lane's entry of the start table and the first live
// block's coefficients.
template <int NP>
__device__ __forceinline__ void m_begin(MState<NP> &st, double2 *stash, int i,
                                        const int *__restrict__ mval,
                                        const long long *__restrict__ soff,
                                        const long long *__restrict__ boff16, int lmax,
                                        const LiveTab &lt, const double *__restrict__ Asb,
                                        const float *__restrict__ Bg, int pb, int lane)
{
    st.i = i;
    const long long e = (long long)i * lt.np + pb * 64 + lane;
    const double2 v = lt.st[e];
    st.l.je = lt.je[e];
    const int jr = ((CIp)(lt.jr + (long long)i * lt.nb))[pb];
    const int len = lmax - ((CIp)mval)[i] + 1;
    st.nblk = (len + kBlk - 1) / kBlk;
    st.q0 = (jr & 0xffff) * kLiveRows / kBlk;
    st.hi8 = (int)((unsigned)jr >> 16) * kLiveRows;
    st.Am = Asb + ((CLp)soff)[i] * kSuperRows;
    st.Bm = Bg + ((CLp)boff16)[i] * (NP * 64) + lane;
    st.l.ua = 0.0;
    st.l.ub = 0.0;
    *stash = v;
    if (st.q0 < st.nblk) {
        scalar_rows<kBlk>(st.a, (CDp)st.Am + st.q0 * kBlk);
        st.load(st.B, st.q0);
    }
}

template <int NP>
__device__ __forceinline__ void m_compute(MState<NP> &st, const double2 *stash, Sums<NP> &tot)
{
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        tot.e[p] = v4f{};
        tot.o[p] = v4f{};
    }
    for (int q = st.q0; q < st.nblk;) {
        const int end = min((q / kSuper + 1) * kSuper, st.nblk);   // of the super-block
        Sums<NP> acc;
        // the look-ahead stays at the m's last block
        block16<NP, true>(st, stash, q, min(q + 1, st.nblk - 1), acc);
        for (++q; q < end; ++q)
            block16<NP, false>(st, stash, q, min(q + 1, st.nblk - 1), acc);
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            tot.e[p] += acc.e[p];
            tot.o[p] += acc.o[p];
        }
    }
}

// Delta of one m (the maps of a ring contiguous, see m_store of the other forms): the lane
// holds its pair's parity sums of every map.  North (E + O) and south (E - O)
// are formed exactly in FP64 and rounded once to FP32.
template <int NP>
__device__ __forceinline__ void store_delta(const Sums<NP> &tot, int i,
                                            float2 *__restrict__ delta,
                                            const PairDesc *__restrict__ pairs, int npairs, int p,
                                            int map0, int nmaps, const DeltaLayout &dl, bool full)
{
    if (p >= npairs) return;
    const PairDesc d = pairs[p];
    if (!full && i >= d.ilim32) return;   // dead on the ring, not read
    const int rs = d.rs >= 0 ? d.rs : d.rn;
    float2 *__restrict__ dn = delta + dl.row(d.rn) + i * dl.mstride(d.rn);
    float2 *__restrict__ ds = delta + dl.row(rs) + i * dl.mstride(rs);
#pragma unroll
    for (int b = 0; b < NP; ++b) {
        const int m0 = map0 + 2 * b;
        float2 n[2], so[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const double er = tot.e[b][2 * k], ei = tot.e[b][2 * k + 1];
            const double orr = tot.o[b][2 * k], oi = tot.o[b][2 * k + 1];
            n[k] = make_float2((float)(er + orr), (float)(ei + oi));
            so[k] = make_float2((float)(er - orr), (float)(ei - oi));
        }
        if (m0 + 1 < nmaps && (nmaps & 1) == 0) {
            *reinterpret_cast<float4 *>(dn + m0) = make_float4(n[0].x, n[0].y, n[1].x, n[1].y);
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

// Groups of 2 NP maps from map0 on.
template <int NP, int W>
__global__ __launch_bounds__(64 * W) void k_legendre_mfma_f32(
    const PairDesc *__restrict__ pairs, int npairs, LiveTab lt, int pblocks,
    const int *__restrict__ mval, const long long *__restrict__ soff,
    const long long *__restrict__ boff16, int nm, int nmpairs, int lmax,
    const double *__restrict__ Asb, const float *__restrict__ Bp, long long nblocks,
    float2 *__restrict__ delta, DeltaLayout dl, int map0, int nmaps, int groups, int full)
{
    __shared__ double2 start[64 * W];
    // XCD x takes the m-pairs q = x mod 8 (see the FP64 kernel)
    const int xcd = (int)(blockIdx.x % 8);
    const int w = xcd_wave<W>();
    const int pb = w % pblocks;
    const int rest = w / pblocks;
    const int grp = rest % groups;
    const int q = xcd + 8 * (rest / groups);
    if (q >= nmpairs) return;
    const int lane = (int)threadIdx.x & 63;
    double2 *stash = start + threadIdx.x;
    const float *Bg = Bp + (long long)grp * nblocks * (NP * 64);
    const int m0 = map0 + grp * 2 * NP;
    const int p = pb * 64 + lane;
    MState<NP> st;
    Sums<NP> tot;
    st.l.x = pairs[p].x;
    m_begin(st, stash, q, mval, soff, boff16, lmax, lt, Asb, Bg, pb, lane);
    m_compute(st, stash, tot);
    const int i1 = st.i;
    const int i2 = nm - 1 - q;
    const bool two = i2 != q;
    // the second m's loads go out before the first one's stores
    if (two) m_begin(st, stash, i2, mval, soff, boff16, lmax, lt, Asb, Bg, pb, lane);
    store_delta(tot, i1, delta, pairs, npairs, p, m0, nmaps, dl, full != 0);
    if (two) {
        m_compute(st, stash, tot);
        store_delta(tot, st.i, delta, pairs, npairs, p, m0, nmaps, dl, full != 0);
    }
}

// Calls f(first map, groups, map pairs per group) for the plan's maps in
// groups of 16 and for the maps left over.
template <typename F>
hipError_t for_groups(const sht_plan_s *p, const F &f)
{
    const int groups = p->nmaps / (2 * kMaxPairs), rest = p->nmaps - groups * 2 * kMaxPairs;
    hipError_t e = hipSuccess;
    if (groups > 0) e = f(0, groups, kMaxPairs);
    if (e == hipSuccess && rest > 0) e = f(groups * 2 * kMaxPairs, 1, (rest + 1) / 2);
    return e;
}

// Floats of the packed B before map `first` (a multiple of 16).
size_t b_offset(const sht_plan_s *p, int first)
{
    return (size_t)(first / 2) * (size_t)p->nblk16 * 64;
}

template <int NP>
hipError_t launch_group(const sht_plan_s *p, const float *Bp, float2 *delta, int first, int groups,
                        bool full, hipStream_t st)
{
    const int pblocks = (p->npairs + 63) / 64;
    const int nmpairs = (p->nm + 1) / 2;
    const int W = waves_per_group(p, (long long)nmpairs * pblocks * groups);
    const long long xcd = (long long)((nmpairs + 7) / 8) * pblocks * groups;   // an XCD's waves
    const long long grid = 8 * ((xcd + W - 1) / W);
    if (grid <= 0 || grid > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    const auto kern = W == 4 ? k_legendre_mfma_f32<NP, 4> : k_legendre_mfma_f32<NP, 1>;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3((unsigned)(64 * W)), 0, st, p->d_pairs,
                       p->npairs, p->live32, pblocks, p->d_mval, p->d_soff, p->d_boff16, p->nm,
                       nmpairs, p->lmax, p->d_Asb, Bp + b_offset(p, first), p->nblk16, delta,
                       delta_blocked_maps(p->nm, p->nrings, p->nmaps), first, p->nmaps, groups, full ? 1 : 0);
    return hipGetLastError();
}

}  // namespace

size_t mfma_bf_bytes(const sht_plan_s *p)
{
    return (size_t)((p->nmaps + 1) / 2) * (size_t)p->nblk16 * 64 * sizeof(float);
}

hipError_t launch_prescale_f32(const sht_plan_s *p, const double *alm, float *Bp, hipStream_t st)
{
    const long long m0len = (p->mval[0] == 0) ? (p->lmax + 1) : 0;
    if (p->nblk16 <= 0 || p->nblk16 > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    return for_groups(p, [&](int first, int groups, int np) {
        dim3 grid((unsigned)((p->nblk16 + kPreBlocks - 1) / kPreBlocks), (unsigned)groups);
        hipLaunchKernelGGL(k_prescale_f32, grid, dim3(256), 0, st,
                           reinterpret_cast<const double2 *>(alm) + first * p->nalm, p->d_cn,
                           p->d_moff, p->d_mval, p->d_boff16, p->d_bm16, p->lmax, p->nalm,
                           p->nblk16, p->nmaps - first, np, m0len, Bp + b_offset(p, first));
        return hipGetLastError();
    });
}

hipError_t launch_legendre_mfma_f32(const sht_plan_s *p, const float *Bp, float2 *delta,
                                    bool full, hipStream_t st)
{
    // the plan's zero-padded coefficient copy has the super-block length of this kernel
    if (f16_super_rows() != kSuperRows) return hipErrorInvalidConfiguration;
    return for_groups(p, [&](int first, int groups, int np) {
        switch (np) {
        case 1: return launch_group<1>(p, Bp, delta, first, groups, full, st);
        case 2: return launch_group<2>(p, Bp, delta, first, groups, full, st);
        case 3: return launch_group<3>(p, Bp, delta, first, groups, full, st);
        case 4: return launch_group<4>(p, Bp, delta, first, groups, full, st);
        case 5: return launch_group<5>(p, Bp, delta, first, groups, full, st);
        case 6: return launch_group<6>(p, Bp, delta, first, groups, full, st);
        case 7: return launch_group<7>(p, Bp, delta, first, groups, full, st);
        case 8: return launch_group<8>(p, Bp, delta, first, groups, full, st);
        default: return hipErrorInvalidValue;
        }
    });
}

}  // namespace sht
