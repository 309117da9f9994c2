// Mixed-precision batched Legendre stage with 3-way split BF16 inputs on
// the matrix cores (gfx950, v_mfma_f32_32x32x16_bf16).
//
// Same contraction as the FP32 form (per m, C_E/O = B_E/O^T Lambda_E/O^T,
// Delta_N = C_E + C_O, Delta_S = C_E - C_O) with every FP32 operand x written
// as x = x_h + x_m + x_l, three BF16 parts, and the product taken as the six
// terms A_h B_h + A_h B_m + A_m B_h + A_h B_l + A_m B_m + A_l B_h; the dropped
// terms are below 2^-23 relative.  The coefficients are split by rounding
// (prescale); the P_lm by truncation, which is exact in FP32 arithmetic:
// x_h = x with the low 16 bits cleared, r = x - x_h (exact), x_m = r with the
// low 16 bits cleared, x_l = r - x_m (exact, at most 8 significant bits), so
// each part is the high half of an FP32 word and two parts pack into one
// dword with one byte permute.  Accumulation is two-level FP32 as in the FP32
// form (64 same-parity terms per first-level block).  The recurrence stays
// FP64 on the vector units.
//
// Fragments.  A 32x32x16 fragment holds, in lanes 0-31, K = 0..7 of its 32
// columns and, in lanes 32-63, K = 8..15.  A lane runs 32 steps of its own
// ring pair; its 16 values of one parity are exchanged across the wave
// halves as FP32 (one v_permlane32_swap per pair of values) and then split,
// which gives the fragments of both column halves.  The coefficient
// fragment is passed first, so the tiles hold the transposed product as in
// the FP32 form, and the same epilogue stores Delta.
//
// Work split.  As in the split-FP16 form: one wave per (64 ring pairs, m-pair,
// 16 maps), two waves per SIMD, nothing shared between waves; each starts at
// its own first live row (live.hip), reads the packed coefficients straight
// into its fragments (from L2) and A_l through scalar registers, and issues
// the products of a parity among the vector work that follows it.
//
// Bound: vector issue (300 vector instructions and 24 MFMA per 32 rows, which
// overlap).  16 maps at l_max 1024 / nside 512: 251 us, the whole transform at
// l_max 4096 / nside 2048 18.2 ms; 340 us and 21.9 ms as workgroups of four
// waves with the coefficients in LDS, every row from l = m on.
#include <type_traits>

#include "mixed_common.h"

namespace sht {
namespace {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

constexpr int kBlkSteps = 32;               // l-rows per block (K = 16 per parity)
// Packed B layout per m block: [parity 2][level 3][half 2][column 32] x 8 bf16.
constexpr int kBlkElems = 2 * 3 * 2 * 32;   // 16-byte elements per block
constexpr int kSuper = 4;                   // blocks per super-block: 64 terms per parity
constexpr int kSuperRows = kSuper * kBlkSteps;

__device__ inline void split3(float x, __bf16 &h, __bf16 &m, __bf16 &l)
{
    h = (__bf16)x;
    const float r1 = x - (float)h;
    m = (__bf16)r1;
    const float r2 = r1 - (float)m;
    l = (__bf16)r2;
}

// a'_lm = c_lm a_lm of up to 16 maps, split and packed per 32-step block.
// One workgroup per kPreBlocks consecutive blocks (bm32: the m of each
// block): the a_lm are read in runs of 32 rows per map (each complex value
// once), split, placed into the packed blocks in LDS, and the blocks are
// written out contiguously.
constexpr int kPreBlocks = 4;

__global__ __launch_bounds__(256) void k_prescale_bf16x3(
    const double2 *__restrict__ alm, const double *__restrict__ cn,
    const long long *__restrict__ moff, const int *__restrict__ mval,
    const long long *__restrict__ boff, const int *__restrict__ bm32, int lmax, long long nalm,
    long long nblocks, int nmaps, long long m0len, v4u *__restrict__ Bb)
{
    __shared__ __attribute__((aligned(16))) __bf16 stage[kPreBlocks * kBlkElems * 8];
    const long long blk0 = (long long)blockIdx.x * kPreBlocks;
    const int nb = (int)min((long long)kPreBlocks, nblocks - blk0);
    const int grp = blockIdx.y;
    const int tid = threadIdx.x;
#pragma unroll
    for (int q = 0; q < kPreBlocks * kBlkSteps * 16 / 256; ++q) {
        const int idx = tid + 256 * q;
        const int b = idx >> 9, mp = (idx >> 5) & 15, rb = idx & 31;   // block, map, row
        if (b < nb) {
            const int i = bm32[blk0 + b];
            const int len = lmax - mval[i] + 1;
            const long long row = (blk0 + b - boff[i]) * kBlkSteps + rb;
            const int map = grp * 16 + mp;
            float xr = 0.0f, xi = 0.0f;
            if (row < len && map < nmaps) {
                const long long e = moff[i] + row;
                const double2 a = alm[(long long)map * nalm + e];
                const double c = cn[e];
                xr = (float)(a.x * c);
                xi = (float)((e < m0len) ? 0.0 : a.y * c);
            }
            // row rb = 2 K + parity; K = 8 half + slot
            const int par = rb & 1, kk = rb >> 1, half = kk >> 3, slot = kk & 7;
            __bf16 h, m, l;
            __bf16 *s = stage + b * kBlkElems * 8;
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                split3(c ? xi : xr, h, m, l);
                const int col = 2 * mp + c;
                s[(((par * 3 + 0) * 2 + half) * 32 + col) * 8 + slot] = h;
                s[(((par * 3 + 1) * 2 + half) * 32 + col) * 8 + slot] = m;
                s[(((par * 3 + 2) * 2 + half) * 32 + col) * 8 + slot] = l;
            }
        }
    }
    __syncthreads();
    const v4u *s4 = reinterpret_cast<const v4u *>(stage);
    v4u *o4 = Bb + ((long long)grp * nblocks + blk0) * kBlkElems;
#pragma unroll
    for (int q = 0; q < kPreBlocks * kBlkElems / 256; ++q) {
        const int w = tid + 256 * q;
        if (w < nb * kBlkElems) o4[w] = s4[w];
    }
}

// High halves of two FP32 words: (a >> 16) | (b & 0xffff0000).
__device__ inline unsigned pack_hi(unsigned a, unsigned b)
{
    return __builtin_amdgcn_perm(b, a, 0x07060302u);
}

// Truncation split of 8 FP32 values (K slots 0-7 of a fragment) into the
// packed BF16 fragments of the three parts.
__device__ inline void split_pack(const float (&f)[8], v4u &H, v4u &M, v4u &L)
{
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const float x0 = f[2 * w], x1 = f[2 * w + 1];
        const unsigned u0 = __float_as_uint(x0), u1 = __float_as_uint(x1);
        const float r0 = x0 - __uint_as_float(u0 & 0xffff0000u);
        const float r1 = x1 - __uint_as_float(u1 & 0xffff0000u);
        const unsigned s0 = __float_as_uint(r0), s1 = __float_as_uint(r1);
        const float l0 = r0 - __uint_as_float(s0 & 0xffff0000u);
        const float l1 = r1 - __uint_as_float(s1 & 0xffff0000u);
        H[w] = pack_hi(u0, u1);
        M[w] = pack_hi(s0, s1);
        L[w] = pack_hi(__float_as_uint(l0), __float_as_uint(l1));
    }
}

__device__ __forceinline__ v16f mfma_bf(const v4u &b, const v4u &a, const v16f &c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, b),
                                                   __builtin_bit_cast(v8bf, a), c, 0, 0, 0);
}

// The fragments of one parity of a block (both column halves, three parts)
// and its coefficient parts.
struct Frags {
    v4u H0, M0, L0, H1, M1, L1, B[3];
};

// The 16 same-parity values of this lane (K = 0..15 of its ring pair) ->
// fragments of both column halves.
__device__ __forceinline__ void split_parity(const float (&v)[16], Frags &f)
{
    float f0[8], f1[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) swap_halves(v[t], v[t + 8], f0[t], f1[t]);
    split_pack(f0, f.H0, f.M0, f.L0);
    split_pack(f1, f.H1, f.M1, f.L1);
}

// Products k0..k1 - 1 (of 12) of a parity, against the lane's coefficient
// parts.  ZERO: the first pair starts the sums.
template <int k0, int k1, bool ZERO>
__device__ __forceinline__ void products(const Frags &f, v16f &acc0, v16f &acc1)
{
    if constexpr (k0 < k1) {
        constexpr int t = k0 / 2;   // A_h B_h, A_m B_h, A_h B_m, A_l B_h, A_m B_m, A_h B_l
        constexpr int lev = t == 2 || t == 4 ? 1 : t == 5 ? 2 : 0;
        const v4u &b = f.B[lev];
        if constexpr (k0 & 1) {
            const v4u &a = t == 1 || t == 4 ? f.M1 : t == 3 ? f.L1 : f.H1;
            acc1 = mfma_bf(b, a, ZERO && k0 == 1 ? v16f{} : acc1);
        } else {
            const v4u &a = t == 1 || t == 4 ? f.M0 : t == 3 ? f.L0 : f.H0;
            acc0 = mfma_bf(b, a, ZERO && k0 == 0 ? v16f{} : acc0);
        }
        products<k0 + 1, k1, ZERO>(f, acc0, acc1);
    }
}

// One block of 32 l-rows from row r0 on (see the split-FP16 form).  FIRST:
// nothing is left from the previous block of the super-block, the sums start
// here; SECOND: what is left starts the odd sums.  B: the block's packed
// coefficients (the lane's first); a0: the coefficients of rows r0..r0 + 15
// on entry, of rows rn..rn + 15 on return.
template <bool FIRST, bool SECOND>
__device__ __forceinline__ void block32(Lane &l, const double2 *stash, int r0, int hi8, CDp Am,
                                        int rn, double (&a0)[16], const v4u *__restrict__ B,
                                        Frags &odd, MfmaTiles &acc)
{
    float ve[16], vo[16];
    double a1[16];
    scalars_arrived();
    scalar_rows<16>(a1, Am + r0 + 16);
    __builtin_amdgcn_sched_barrier(0);
    Frags even;
#pragma unroll
    for (int lev = 0; lev < 3; ++lev) even.B[lev] = B[lev * 64];
    enter(l, stash, r0, hi8);
    rows8(l, a0, ve, vo);
    if constexpr (!FIRST) products<0, 3, SECOND>(odd, acc.o0, acc.o1);
    enter(l, stash, r0 + 8, hi8);
    rows8(l, a0 + 8, ve + 4, vo + 4);
    if constexpr (!FIRST) products<3, 6, SECOND>(odd, acc.o0, acc.o1);
    scalars_arrived();
    scalar_rows<16>(a0, Am + rn);
    __builtin_amdgcn_sched_barrier(0);
    enter(l, stash, r0 + 16, hi8);
    rows8(l, a1, ve + 8, vo + 8);
    if constexpr (!FIRST) products<6, 9, SECOND>(odd, acc.o0, acc.o1);
    enter(l, stash, r0 + 24, hi8);
    rows8(l, a1 + 8, ve + 12, vo + 12);
    if constexpr (!FIRST) products<9, 12, SECOND>(odd, acc.o0, acc.o1);
#pragma unroll
    for (int lev = 0; lev < 3; ++lev) odd.B[lev] = B[(3 + lev) * 64];
    split_parity(ve, even);
    products<0, 12, FIRST>(even, acc.e0, acc.e1);
    split_parity(vo, odd);
    // one product to eight vector instructions (8 exchanges, 88 of the split)
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);
    }
}

struct MState {
    int i, nblk, q0;     // blocks of the m, the first one with a live row of the wave
    int hi8;             // the last row at which a pair starts
    const double *Am;    // padded coefficients of the m, per super-block
    const v4u *Bm;       // its packed blocks, the lane's first entry
    Lane l;
    double a[16];
};

// Start of an m: the lane's entry of the start table and the first live
// block's coefficients.
__device__ __forceinline__ void m_begin(MState &st, double2 *stash, int i,
                                        const int *__restrict__ mval,
                                        const long long *__restrict__ boff,
                                        const long long *__restrict__ soff, int lmax,
                                        const LiveTab &lt, const double *__restrict__ Asb,
                                        const v4u *__restrict__ Bg, int pb, int lane)
{
    st.i = i;
    const long long e = (long long)i * lt.np + pb * 64 + lane;
    const double2 v = lt.st[e];
    st.l.je = lt.je[e];
    const int jr = ((CIp)(lt.jr + (long long)i * lt.nb))[pb];
    const int len = lmax - ((CIp)mval)[i] + 1;
    st.nblk = (len + kBlkSteps - 1) / kBlkSteps;
    st.q0 = (jr & 0xffff) * kLiveRows / kBlkSteps;
    st.hi8 = (int)((unsigned)jr >> 16) * kLiveRows;
    st.Am = Asb + ((CLp)soff)[i] * kSuperRows;
    st.Bm = Bg + ((CLp)boff)[i] * kBlkElems + lane;
    st.l.ua = 0.0;
    st.l.ub = 0.0;
    *stash = v;
    if (st.q0 < st.nblk) scalar_rows<16>(st.a, (CDp)st.Am + st.q0 * kBlkSteps);
}

__device__ __forceinline__ void m_compute(MState &st, const double2 *stash, MfmaTiles &tot)
{
    zero_tiles(tot);
    for (int q = st.q0; q < st.nblk;) {
        const int end = min((q / kSuper + 1) * kSuper, st.nblk);   // of the super-block
        Frags odd;
        MfmaTiles acc;
        // the look-ahead stays at the m's last block
        auto step = [&](auto first, auto second) {
            block32<decltype(first)::value, decltype(second)::value>(
                st.l, stash, q * kBlkSteps, st.hi8, (CDp)st.Am,
                min(q + 1, st.nblk - 1) * kBlkSteps, st.a, st.Bm + (long long)q * kBlkElems, odd,
                acc);
            ++q;
        };
        step(std::true_type(), std::false_type());
        if (q < end) {
            step(std::false_type(), std::true_type());
            while (q < end) step(std::false_type(), std::false_type());
            products<0, 12, false>(odd, acc.o0, acc.o1);
        } else {
            products<0, 12, true>(odd, acc.o0, acc.o1);
        }
        add_tiles(tot, acc);
    }
}

template <int W>
__global__ __launch_bounds__(64 * W, 2) void k_legendre_mfma_bf16x3(
    const PairDesc *__restrict__ pairs, int npairs, LiveTab lt, int pblocks,
    const int *__restrict__ mval, const long long *__restrict__ boff,
    const long long *__restrict__ soff, int nm, int nmpairs, int lmax,
    const double *__restrict__ Asb, const v4u *__restrict__ Bb, long long nblocks,
    float2 *__restrict__ delta, DeltaLayout dl, int nmaps, int groups, int full)
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
    const v4u *Bg = Bb + (long long)grp * nblocks * kBlkElems;
    MState st;
    MfmaTiles tot;
    st.l.x = pairs[pb * 64 + lane].x;
    m_begin(st, stash, q, mval, boff, soff, lmax, lt, Asb, Bg, pb, lane);
    m_compute(st, stash, tot);
    const int i1 = st.i;
    const int i2 = nm - 1 - q;
    const bool two = i2 != q;
    if (two) m_begin(st, stash, i2, mval, boff, soff, lmax, lt, Asb, Bg, pb, lane);
    m_store(tot, i1, delta, pairs, npairs, pb, grp, nmaps, dl, full != 0, lane);
    if (two) {
        m_compute(st, stash, tot);
        m_store(tot, st.i, delta, pairs, npairs, pb, grp, nmaps, dl, full != 0, lane);
    }
}

}  // namespace

size_t bf16_bytes(const sht_plan_s *p)
{
    const size_t groups = (size_t)((p->nmaps + 15) / 16);
    return groups * (size_t)p->nblk32 * kBlkElems * 16;
}

hipError_t launch_prescale_bf16x3(const sht_plan_s *p, const double *alm, void *Bb,
                                  hipStream_t st)
{
    const long long m0len = (p->mval[0] == 0) ? (p->lmax + 1) : 0;
    const int groups = (p->nmaps + 15) / 16;
    const long long nblocks = p->nblk32;
    const long long nwg = (nblocks + kPreBlocks - 1) / kPreBlocks;
    if (nwg <= 0 || nwg > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(k_prescale_bf16x3, dim3((unsigned)nwg, (unsigned)groups), dim3(256), 0, st,
                       reinterpret_cast<const double2 *>(alm), p->d_cn, p->d_moff, p->d_mval,
                       p->d_boff, p->d_bm32, p->lmax, p->nalm, nblocks, p->nmaps, m0len,
                       reinterpret_cast<v4u *>(Bb));
    return hipGetLastError();
}

hipError_t launch_legendre_mfma_bf16x3(const sht_plan_s *p, const void *Bb, float2 *delta,
                                       bool full, hipStream_t st)
{
    const int pblocks = (p->npairs + 63) / 64;
    const int nmpairs = (p->nm + 1) / 2;
    const int groups = (p->nmaps + 15) / 16;
    const int W = waves_per_group(p, (long long)nmpairs * pblocks * groups);
    const long long xcd = (long long)((nmpairs + 7) / 8) * pblocks * groups;   // an XCD's waves
    const long long grid = 8 * ((xcd + W - 1) / W);
    if (grid <= 0 || grid > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    // the plan's zero-padded coefficient copy has the super-block length of this kernel
    if (f16_super_rows() != kSuperRows) return hipErrorInvalidConfiguration;
    const auto kern = W == 4 ? k_legendre_mfma_bf16x3<4> : k_legendre_mfma_bf16x3<1>;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3((unsigned)(64 * W)), 0, st,
                       p->d_pairs, p->npairs, p->live32, pblocks, p->d_mval, p->d_boff, p->d_soff,
                       p->nm, nmpairs, p->lmax, p->d_Asb, reinterpret_cast<const v4u *>(Bb),
                       p->nblk32, delta, delta_blocked_maps(p->nm, p->nrings, p->nmaps), p->nmaps, groups, full ? 1 : 0);
    return hipGetLastError();
}

}  // namespace sht
