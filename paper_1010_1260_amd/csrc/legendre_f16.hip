// Mixed-precision batched Legendre stage with 2-way split FP16 inputs on the
// matrix cores (gfx950, v_mfma_f32_32x32x16_f16).
//
// Same contraction as the FP32 form (per m, C_E/O = B_E/O^T Lambda_E/O^T,
// Delta_N = C_E + C_O, Delta_S = C_E - C_O).  Every FP32 operand x is written
// as x = x_h + x_l with x_h = x rounded to FP16 and x_l = (x - x_h) rounded
// to FP16 (the difference is exact in FP32), about 22 significant bits
// together; the product is taken as the three terms
// A_h B_h + A_h B_l + A_l B_h, the dropped A_l B_l being below 2^-21
// relative.  Products of FP16 numbers are exact in FP32, and accumulation
// is two-level FP32 as in the FP32 form (64 same-parity terms per
// first-level block).  The recurrence stays FP64 on the vector units.
//
// Range.  FP16 carries 5 exponent bits, so both operands are moved into its
// range by powers of two (exact).  The P_lm values: u = P_lm / c_lm is below
// 2^8.75 for l <= 16383 at scaled exponent k = 0 (addition theorem and the
// smallest c_lm), and the seed is multiplied by 2^6, so every matrix operand
// stays below 2^15.  The coefficients: per map and 128-row super-block the
// prescale picks 2^e with the largest magnitude in [2^14, 2^15).  The
// first-level sums of a super-block are multiplied by 2^-(e+6) as they are
// added into the second-level sums (one FMA per entry, as many instructions
// as the plain add).  Past an m's last row the recurrence coefficients are
// zero (a padded copy of the table per super-block), so u stays bounded
// there and its product with the zero coefficients is zero, never 0 * inf.
//
// Fragments.  A 32x32x16 fragment holds K = 0..7 of its 32 columns in lanes
// 0-31 and K = 8..15 in lanes 32-63; a lane's 16 same-parity values are
// exchanged across the wave halves as FP32 and then split (one packed
// conversion per two values, one mixed-precision FMA per residual, one packed
// conversion per two residuals).
//
// Work split.  One wave per (64 ring pairs, m-pair, 16 maps), two waves per
// SIMD.  The waves share nothing: each reads the packed coefficients straight
// into its fragments (16 bytes per lane, from L2, a block ahead) and A_l
// through scalar registers, starts at its own first live row (live.hip) and
// runs the recurrence alone while every operand would be zero in FP16 (below
// 2^-32).  FP16 matrix instructions run beside FP64 vector ones (measured: an
// MFMA and eight FP64 FMAs 45 cycles, alone 36 and 36), so the products of a
// parity are issued among the vector work that follows it.
//
// Bound: vector issue at the power limit.  204 vector instructions and 12 MFMA
// per 32 rows.  l_max 4096 / nside 2048, 16 maps: 7.71 ms (counted: vector issue
// on 73% of the cycles, at 1.8-2.0 GHz); 10.8 ms as workgroups of four waves that
// shared the coefficients in LDS with a barrier per super-block, every row
// from l = m on; 8.63 ms so with the live rows and the interleaved products,
// 8.14 ms with independent waves.
#include <type_traits>

#include "mixed_common.h"

namespace sht {
namespace {

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));

constexpr int kWaves = 4;                   // waves of a prescale workgroup
constexpr int kBlkSteps = 32;               // l-rows per block (K = 16 per parity)
// Packed B layout per block: [parity 2][level 2][half 2][column 32] x 8 fp16.
constexpr int kBlkElems = 2 * 2 * 2 * 32;   // 16-byte elements per block
constexpr int kSuper = 4;                   // blocks per super-block: 64 terms per parity
constexpr int kSuperRows = kSuper * kBlkSteps;
constexpr int kScaleElems = 4;              // 16 FP32 inverse scales (one per map)
constexpr int kSuperElems = kSuper * kBlkElems + kScaleElems;
constexpr double kPScale = 0x1p6;           // P_lm operands are u * 2^6

// Two FP32 values rounded to FP16 (round to nearest even), packed.  The
// empty asm keeps the compiler from re-deriving either half from x (it would
// convert each value again).
__device__ inline unsigned pk_f16(float a, float b)
{
    const v2h h = {(_Float16)a, (_Float16)b};
    unsigned u = __builtin_bit_cast(unsigned, h);
    asm("" : "+v"(u));
    return u;
}

// x - (float)low / high half of h, exact (one mixed-precision FMA).
__device__ inline float res_lo(unsigned h, float x)
{
    float r;
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(r) : "v"(h), "v"(x));
    return r;
}
__device__ inline float res_hi(unsigned h, float x)
{
    float r;
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r)
        : "v"(h), "v"(x));
    return r;
}

// 8 FP32 values (K slots 0-7 of a fragment) -> packed FP16 high and low parts.
__device__ inline void split_pack(const float (&f)[8], v4u &H, v4u &L)
{
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const unsigned h = pk_f16(f[2 * w], f[2 * w + 1]);
        H[w] = h;
        L[w] = pk_f16(res_lo(h, f[2 * w]), res_hi(h, f[2 * w + 1]));
    }
}

__device__ __forceinline__ v16f mfma_h(const v4u &b, const v4u &a, const v16f &c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, b),
                                                  __builtin_bit_cast(v8h, a), c, 0, 0, 0);
}

// a'_lm = c_lm a_lm of up to 16 maps for one 128-row super-block of an m:
// scaled per map by 2^e (largest magnitude into [2^14, 2^15)), split into
// FP16 parts and packed; the inverse scales 2^-(e+6) follow the blocks.
// One workgroup per super-block (sbm: the m of each super-block); thread
// item idx = tid + 256 q is (map idx / 128, row idx % 128), so the a_lm of
// a map are read in runs of 128 rows.
__global__ __launch_bounds__(256) void k_prescale_f16x2(
    const double2 *__restrict__ alm, const double *__restrict__ cn,
    const long long *__restrict__ moff, const int *__restrict__ mval,
    const long long *__restrict__ soff, const int *__restrict__ sbm, int lmax, long long nalm,
    long long nsuper, int nmaps, long long m0len, v4u *__restrict__ Bb)
{
    __shared__ __attribute__((aligned(16))) _Float16 stage[kSuperElems * 8];
    __shared__ float wmax[kWaves][8];
    __shared__ int wexp[16];
    const long long s = blockIdx.x;
    const int grp = blockIdx.y;
    const int tid = threadIdx.x;
    const int i = sbm[s];
    const int len = lmax - mval[i] + 1;
    const long long row0 = (s - soff[i]) * kSuperRows;
    double2 v[8];
    float mx[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int idx = tid + 256 * q;
        const int mp = idx >> 7, rb = idx & 127;
        const long long row = row0 + rb;
        const int map = grp * 16 + mp;
        double2 b = make_double2(0.0, 0.0);
        if (row < len && map < nmaps) {
            const long long e = moff[i] + row;
            const double2 a = alm[(long long)map * nalm + e];
            const double c = cn[e];
            b.x = a.x * c;
            b.y = (e < m0len) ? 0.0 : a.y * c;
        }
        v[q] = b;
        mx[q] = (float)fmax(fabs(b.x), fabs(b.y));   // rounding cannot move a power of two
    }
    // per map (= 2 q + wave / 2): max over its 128 rows, two waves of 64
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        float m = mx[q];
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
        mx[q] = m;
    }
    const int wave = tid >> 6;
    if ((tid & 63) == 0) {
#pragma unroll
        for (int q = 0; q < 8; ++q) wmax[wave][q] = mx[q];
    }
    __syncthreads();
    if (tid < 16) {
        const int q = tid >> 1, w0 = 2 * (tid & 1);
        const float m = fmaxf(wmax[w0][q], wmax[w0 + 1][q]);
        int e = 0;
        if (m > 0.0f) {
            int E;
            (void)frexpf(m, &E);          // m < 2^E
            e = min(max(15 - E, -120), 120);
        }
        wexp[2 * q + (tid & 1)] = e;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int idx = tid + 256 * q;
        const int mp = idx >> 7, rb = idx & 127;
        const int map = 2 * q + (tid >> 7);   // = mp
        const double sc = ldexp(1.0, wexp[map]);
        const int blk = rb >> 5, r32 = rb & 31;
        const int par = r32 & 1, kk = r32 >> 1, half = kk >> 3, slot = kk & 7;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const float x = (float)((c ? v[q].y : v[q].x) * sc);
            const _Float16 h = (_Float16)x;
            const _Float16 l = (_Float16)(x - (float)h);
            const int col = 2 * mp + c;
            _Float16 *st = stage + (size_t)blk * kBlkElems * 8;
            st[(((par * 2 + 0) * 2 + half) * 32 + col) * 8 + slot] = h;
            st[(((par * 2 + 1) * 2 + half) * 32 + col) * 8 + slot] = l;
        }
    }
    if (tid < 16)
        reinterpret_cast<float *>(stage + kSuper * kBlkElems * 8)[tid] =
            (float)ldexp(1.0, -(wexp[tid] + 6));
    __syncthreads();
    const v4u *s4 = reinterpret_cast<const v4u *>(stage);
    v4u *o4 = Bb + ((long long)grp * nsuper + s) * kSuperElems;
#pragma unroll
    for (int q = 0; q < kSuper * kBlkElems / 256; ++q) o4[tid + 256 * q] = s4[tid + 256 * q];
    if (tid < kScaleElems) o4[kSuper * kBlkElems + tid] = s4[kSuper * kBlkElems + tid];
}

// The fragments of one parity of a block (both column halves, high and low
// parts) and its coefficient parts.
struct Frags {
    v4u H0, L0, H1, L1, B0, B1;
};

// The 16 same-parity values of this lane (K = 0..15 of its ring pair) ->
// fragments of both column halves.
__device__ __forceinline__ void split_parity(const float (&v)[16], Frags &f)
{
    float f0[8], f1[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) swap_halves(v[t], v[t + 8], f0[t], f1[t]);
    split_pack(f0, f.H0, f.L0);
    split_pack(f1, f.H1, f.L1);
}

// The k-th (0..5) of the products of a parity, against the lane's
// coefficient parts.  ZERO: the first pair starts the sums.
template <int k, bool ZERO>
__device__ __forceinline__ void product(const Frags &f, v16f &acc0, v16f &acc1)
{
    if constexpr (k == 0) acc0 = mfma_h(f.B0, f.H0, ZERO ? v16f{} : acc0);
    if constexpr (k == 1) acc1 = mfma_h(f.B0, f.H1, ZERO ? v16f{} : acc1);
    if constexpr (k == 2) acc0 = mfma_h(f.B0, f.L0, acc0);
    if constexpr (k == 3) acc1 = mfma_h(f.B0, f.L1, acc1);
    if constexpr (k == 4) acc0 = mfma_h(f.B1, f.H0, acc0);
    if constexpr (k == 5) acc1 = mfma_h(f.B1, f.H1, acc1);
}

template <bool ZERO>
__device__ __forceinline__ void all_products(const Frags &f, v16f &acc0, v16f &acc1)
{
    product<0, ZERO>(f, acc0, acc1);
    product<1, ZERO>(f, acc0, acc1);
    product<2, ZERO>(f, acc0, acc1);
    product<3, ZERO>(f, acc0, acc1);
    product<4, ZERO>(f, acc0, acc1);
    product<5, ZERO>(f, acc0, acc1);
}

__device__ __forceinline__ void rows8_quiet(Lane &l, const double *a)
{
#pragma unroll
    for (int t = 0; t < 8; t += 2) {
        l.ua = fma(a[t] * l.x, l.ub, -l.ua);
        l.ub = fma(a[t + 1] * l.x, l.ua, -l.ub);
    }
}

// The coefficient parts of a block: [parity][level], one 16-byte load each,
// straight in the fragment layout.
struct BParts {
    v4u b[2][2];

    __device__ __forceinline__ void load(const v4u *__restrict__ Bl)
    {
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int lev = 0; lev < 2; ++lev) b[p][lev] = Bl[(p * 2 + lev) * 64];
    }
};

// One block of 32 l-rows from row r0 on.  The matrix core works beside the
// vector units: the products of a block's odd parity are issued among the
// next block's recurrence, those of its even parity among the conversions
// of its odd values.  FIRST: nothing is left from the previous block of the
// super-block, the sums start here; SECOND: what is left starts the odd sums.
// On entry a0 holds the coefficients of rows r0..r0 + 15 and B the block's
// parts (asked for a half block and a block ahead); on return those of rows rn
// on and of the block at Bn.
template <bool FIRST, bool SECOND>
__device__ __forceinline__ void block32(Lane &l, const double2 *stash, int r0, int hi8, CDp Am,
                                        int rn, double (&a0)[16], const v4u *__restrict__ Bn,
                                        BParts &B, Frags &odd, MfmaTiles &acc)
{
    float ve[16], vo[16];
    double a1[16];
    scalars_arrived();
    scalar_rows<16>(a1, Am + r0 + 16);
    __builtin_amdgcn_sched_barrier(0);
    Frags even;
    even.B0 = B.b[0][0];
    even.B1 = B.b[0][1];
    const v4u bo0 = B.b[1][0], bo1 = B.b[1][1];
    B.load(Bn);
    enter(l, stash, r0, hi8, kPScale);
    rows8(l, a0, ve, vo);
    if constexpr (!FIRST) { product<0, SECOND>(odd, acc.o0, acc.o1); product<1, SECOND>(odd, acc.o0, acc.o1); }
    enter(l, stash, r0 + 8, hi8, kPScale);
    rows8(l, a0 + 8, ve + 4, vo + 4);
    if constexpr (!FIRST) product<2, SECOND>(odd, acc.o0, acc.o1);
    scalars_arrived();
    scalar_rows<16>(a0, Am + rn);
    __builtin_amdgcn_sched_barrier(0);
    enter(l, stash, r0 + 16, hi8, kPScale);
    rows8(l, a1, ve + 8, vo + 8);
    if constexpr (!FIRST) { product<3, SECOND>(odd, acc.o0, acc.o1); product<4, SECOND>(odd, acc.o0, acc.o1); }
    enter(l, stash, r0 + 24, hi8, kPScale);
    rows8(l, a1 + 8, ve + 12, vo + 12);
    if constexpr (!FIRST) product<5, SECOND>(odd, acc.o0, acc.o1);
    split_parity(ve, even);
    all_products<FIRST>(even, acc.e0, acc.e1);
    split_parity(vo, odd);
    odd.B0 = bo0;
    odd.B1 = bo1;
    // one product to seven vector instructions (8 exchanges, 32 conversions)
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 7, 0);
    }
}

// tot += acc * (inverse scale of the entry's map).  Entry r of a lane's
// tile row set is row 8 (r/4) + 4 hi + r%4 = 2 map + Re/Im, so the lane's
// maps are 4 j + 2 hi + {0, 1}, j = 0..3.
struct Scales {
    float2 s[4];

    __device__ __forceinline__ void load(const v4u *__restrict__ Bs, int hi)
    {
        const float2 *p = reinterpret_cast<const float2 *>(Bs + kSuper * kBlkElems) + hi;
#pragma unroll
        for (int j = 0; j < 4; ++j) s[j] = p[2 * j];
    }
};

__device__ __forceinline__ void add_tiles_scaled(MfmaTiles &tot, const MfmaTiles &acc,
                                                 const Scales &sc)
{
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const float f = (r & 2) ? sc.s[r >> 2].y : sc.s[r >> 2].x;
        tot.e0[r] = fmaf(acc.e0[r], f, tot.e0[r]);
        tot.e1[r] = fmaf(acc.e1[r], f, tot.e1[r]);
        tot.o0[r] = fmaf(acc.o0[r], f, tot.o0[r]);
        tot.o1[r] = fmaf(acc.o1[r], f, tot.o1[r]);
    }
}

// A block whose operands would all be zero: the recurrence alone.
__device__ __forceinline__ void block32_quiet(Lane &l, const double2 *stash, int r0, int hi8,
                                              CDp Am, int rn, double (&a0)[16])
{
    double a1[16];
    scalars_arrived();
    scalar_rows<16>(a1, Am + r0 + 16);
    __builtin_amdgcn_sched_barrier(0);
    enter(l, stash, r0, hi8, kPScale);
    rows8_quiet(l, a0);
    enter(l, stash, r0 + 8, hi8, kPScale);
    rows8_quiet(l, a0 + 8);
    scalars_arrived();
    scalar_rows<16>(a0, Am + rn);
    __builtin_amdgcn_sched_barrier(0);
    enter(l, stash, r0 + 16, hi8, kPScale);
    rows8_quiet(l, a1);
    enter(l, stash, r0 + 24, hi8, kPScale);
    rows8_quiet(l, a1 + 8);
}

struct MState {
    int i, nblk, q0;     // blocks of the m, the first one with a live row of the wave,
    int q1;              // and the first one with an operand that is not zero
    int hi8;             // the last row at which a pair starts
    const double *Am;    // padded coefficients of the m, per super-block
    const v4u *Bm;       // its packed blocks
    Lane l;
    double a[16];
    BParts B;

    __device__ __forceinline__ const v4u *block(int q) const
    {
        return Bm + (long long)(q / kSuper) * kSuperElems + (q % kSuper) * kBlkElems;
    }
};

// Start of an m: the lane's entry of the start table and the first live
// block's coefficients.
__device__ __forceinline__ void m_begin(MState &st, double2 *stash, int i,
                                        const int *__restrict__ mval,
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
    const long long so = ((CLp)soff)[i];
    st.nblk = (len + kBlkSteps - 1) / kBlkSteps;
    st.q0 = (jr & 0xffff) * kLiveRows / kBlkSteps;
    st.hi8 = (int)((unsigned)jr >> 16) * kLiveRows;
    // jq is read as half of an aligned word
    const long long o = (long long)i * lt.nb + pb;
    const int w = ((CIp)lt.jq)[o >> 1];
    st.q1 = ((o & 1) ? (int)((unsigned)w >> 16) : (w & 0xffff)) * kLiveRows / kBlkSteps;
    st.Am = Asb + so * kSuperRows;
    st.Bm = Bg + so * kSuperElems;
    st.l.ua = 0.0;
    st.l.ub = 0.0;
    *stash = v;
    if (st.q1 < st.nblk) {
        scalar_rows<16>(st.a, (CDp)st.Am + st.q0 * kBlkSteps);
        st.B.load(st.block(st.q1) + lane);
    }
}

__device__ __forceinline__ void m_compute(MState &st, const double2 *stash, int lane,
                                          MfmaTiles &tot)
{
    zero_tiles(tot);
    if (st.q1 >= st.nblk) return;
    const CDp Am = (CDp)st.Am;
    for (int q = st.q0; q < st.q1; ++q)
        block32_quiet(st.l, stash, q * kBlkSteps, st.hi8, Am, (q + 1) * kBlkSteps, st.a);
    for (int q = st.q1; q < st.nblk;) {
        const int end = min((q / kSuper + 1) * kSuper, st.nblk);   // of the super-block
        Scales sc;
        sc.load(st.block(q & ~(kSuper - 1)), lane >> 5);
        Frags odd;
        MfmaTiles acc;
        // the look-ahead stays at the m's last block
        auto step = [&](auto first, auto second) {
            const int qn = min(q + 1, st.nblk - 1);
            block32<decltype(first)::value, decltype(second)::value>(
                st.l, stash, q * kBlkSteps, st.hi8, Am, qn * kBlkSteps, st.a,
                st.block(qn) + lane, st.B, odd, acc);
            ++q;
        };
        step(std::true_type(), std::false_type());
        if (q < end) {
            step(std::false_type(), std::true_type());
            while (q < end) step(std::false_type(), std::false_type());
            all_products<false>(odd, acc.o0, acc.o1);
        } else {
            all_products<true>(odd, acc.o0, acc.o1);
        }
        add_tiles_scaled(tot, acc, sc);
    }
}

// One wave per (64 ring pairs, m-pair, 16 maps), nothing shared between waves:
// no barrier, and a wave's dead rows cost it nothing.
template <int W>
__global__ __launch_bounds__(64 * W, 2) void k_legendre_mfma_f16x2(
    const PairDesc *__restrict__ pairs, int npairs, LiveTab lt, int pblocks,
    const int *__restrict__ mval, const long long *__restrict__ soff, int nm, int nmpairs,
    int lmax, const double *__restrict__ Asb, const v4u *__restrict__ Bb, long long nsuper,
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
    const v4u *Bg = Bb + (long long)grp * nsuper * kSuperElems;
    MState st;
    MfmaTiles tot;
    st.l.x = pairs[pb * 64 + lane].x;
    m_begin(st, stash, q, mval, soff, lmax, lt, Asb, Bg, pb, lane);
    m_compute(st, stash, lane, tot);
    const int i1 = st.i;
    const int i2 = nm - 1 - q;
    const bool two = i2 != q;
    if (two) m_begin(st, stash, i2, mval, soff, lmax, lt, Asb, Bg, pb, lane);
    m_store(tot, i1, delta, pairs, npairs, pb, grp, nmaps, dl, full != 0, lane);
    if (two) {
        m_compute(st, stash, lane, tot);
        m_store(tot, st.i, delta, pairs, npairs, pb, grp, nmaps, dl, full != 0, lane);
    }
}

}  // namespace

int f16_super_rows() { return kSuperRows; }

size_t f16_bytes(const sht_plan_s *p)
{
    const size_t groups = (size_t)((p->nmaps + 15) / 16);
    return groups * (size_t)p->nsuper * kSuperElems * 16;
}

hipError_t launch_prescale_f16x2(const sht_plan_s *p, const double *alm, void *Bb,
                                 hipStream_t st)
{
    const long long m0len = (p->mval[0] == 0) ? (p->lmax + 1) : 0;
    const int groups = (p->nmaps + 15) / 16;
    if (p->nsuper <= 0 || p->nsuper > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(k_prescale_f16x2, dim3((unsigned)p->nsuper, (unsigned)groups), dim3(256),
                       0, st, reinterpret_cast<const double2 *>(alm), p->d_cn, p->d_moff,
                       p->d_mval, p->d_soff, p->d_sbm, p->lmax, p->nalm, p->nsuper, p->nmaps,
                       m0len, reinterpret_cast<v4u *>(Bb));
    return hipGetLastError();
}

hipError_t launch_legendre_mfma_f16x2(const sht_plan_s *p, const void *Bb, float2 *delta,
                                      bool full, hipStream_t st)
{
    const int pblocks = (p->npairs + 63) / 64;
    const int nmpairs = (p->nm + 1) / 2;
    const int groups = (p->nmaps + 15) / 16;
    const int W = waves_per_group(p, (long long)nmpairs * pblocks * groups);
    const long long xcd = (long long)((nmpairs + 7) / 8) * pblocks * groups;   // an XCD's waves
    const long long grid = 8 * ((xcd + W - 1) / W);
    if (grid <= 0 || grid > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    const auto kern = W == 4 ? k_legendre_mfma_f16x2<4> : k_legendre_mfma_f16x2<1>;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3((unsigned)(64 * W)), 0, st,
                       p->d_pairs, p->npairs, p->live32, pblocks, p->d_mval, p->d_soff, p->nm,
                       nmpairs, p->lmax, p->d_Asb, reinterpret_cast<const v4u *>(Bb), p->nsuper,
                       delta, delta_blocked_maps(p->nm, p->nrings, p->nmaps), p->nmaps, groups, full ? 1 : 0);
    return hipGetLastError();
}

}  // namespace sht
