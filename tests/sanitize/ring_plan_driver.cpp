// Host-side checks of the ring planning (sht_internal.h), under the
// sanitizers like plan_driver.cpp: the complex128 Bluestein classes, their LDS
// at every number of live modes that the plan admits, the block layouts of
// Delta, and the share of rings that an XCD takes.
#include <cstdio>
#include <set>
#include <vector>

#include "sht_internal.h"

static int fail = 0;
#define CHECK(c)                                                       \
    do {                                                               \
        if (!(c) && fail++ < 20) std::fprintf(stderr, "line %d: %s\n", __LINE__, #c); \
    } while (0)

// convolution lengths of every class and the LDS of their rings
static int blue64_classes()
{
    int lengths = 0;
    for (int q = 0; q < sht::kNumBlue64; ++q) {
        const int nt = sht::kBlue64Threads[q], maxn = sht::kBlue64MaxN[q];
        sht::RingLds cls = {};   // the class: every admitted ring together
        for (int nb = 2; nb <= maxn + 8; ++nb) {
            unsigned long long rads = 0;
            const int np = sht::blue_radices(nb, &rads, nt, maxn, true);
            if (np == 0) continue;
            ++lengths;
            CHECK(nb <= maxn);
            long long prod = 1;
            for (int p = 0; p < np; ++p) {
                const int R = (int)((rads >> (5 * p)) & 31);
                CHECK(R == 8 || R == 4 || R == 2 || R == 7 || R == 5 || R == 3);
                CHECK(nb / R <= nt);   // one butterfly per thread
                prod *= R;
            }
            CHECK(prod == nb);
            CHECK(5 * np <= 64);
            // half lengths h = 2 len with 2 len - 1 <= nb
            for (int h = 2; h <= nb + 1; h += 2) {
                if (h > 64 && h < nb / 2) continue;
                for (int mlive = -1; mlive <= SHT_MAX_LMAX; mlive += 64) {
                    if (!sht::blue64_holds(mlive)) continue;
                    sht::RingLds l = {};
                    sht::blue_lds_add(l, 2 * h, nb, mlive, nt);
                    CHECK(l.fft_entries > sht::fast_pad(h) && l.fft_entries > sht::fast_pad(nb - 1));
                    CHECK(mlive < 0 || l.fft_entries > sht::fast_pad(mlive));
                    CHECK(l.fft_entries > sht::fast_pad(nt - 1));
                    CHECK(l.y_entries > sht::fast_pad(nb - 1));
                    sht::blue_lds_add(cls, 2 * h, nb, mlive, nt);
                    // the class it ends in has the threads and the room
                    const int e = sht::blue64_class(q, 2 * h, nb, mlive);
                    CHECK(e >= q && e < sht::kNumBlue64);
                    sht::RingLds m = {};
                    sht::blue_lds_add(m, 2 * h, nb, mlive, sht::kBlue64Threads[e]);
                    CHECK(e == sht::kNumBlue64 - 1 || m.total() <= sht::kTogetherEntries << e);
                    CHECK(nb <= sht::kBlue64MaxN[e] && sht::kBlue64Threads[e] >= nt);
                }
            }
        }
        CHECK(cls.total() * 16 <= 160 * 1024);
    }
    // the fast paths' modes are bounded alike
    CHECK(!sht::blue64_holds(sht::kFastMaxModes) && sht::blue64_holds(sht::kFastMaxModes - 1));
    return lengths;
}

// every (map, m, ring) has an entry of its own in [0, nmaps nm nrings)
static void one_to_one(const sht::DeltaLayout &dl, int nmaps, int nm, int nrings)
{
    std::vector<char> used((size_t)nmaps * nm * nrings, 0);
    for (int b = 0; b < nmaps; ++b)
        for (int i = 0; i < nm; ++i)
            for (int r = 0; r < nrings; ++r) {
                const long long e = b * dl.map + dl.row(r) + i * dl.mstride(r);
                const bool in = e >= 0 && e < (long long)used.size();
                CHECK(in);
                if (!in) continue;
                CHECK(!used[(size_t)e]);
                used[(size_t)e] = 1;
            }
}

// xcd_share / xcd_item of the ring kernels: ring k of XCD x
static void shares(int count, int nitems, int shift0)
{
    long long grid = 512, items = (long long)count * nitems;
    if (grid > items) grid = items;
    grid = (grid + 7) / 8 * 8;
    const long long per = grid / 8;
    const int s = sht::ring_group(count, nitems, grid, shift0);
    CHECK(s >= 0 && s <= shift0);
    std::set<int> seen;
    long long most = 0;
    for (int x = 0; x < 8; ++x) {
        const int g = 1 << s, all = count >> (s + 3), rest = count - (all << (s + 3)) - (x << s);
        const int n = (all << s) + (rest < 0 ? 0 : rest < g ? rest : g);
        for (int q = 0; q < n; ++q) {
            const int i = ((((q >> s) << 3) + x) << s) + (q & (g - 1));
            CHECK(i < count && seen.insert(i).second);
        }
        if (n > most) most = n;
    }
    CHECK((int)seen.size() == count);
    const long long even = (count + 7) / 8;   // single rings in turn
    CHECK((most * nitems + per - 1) / per <= (even * nitems + per - 1) / per);
}

int main()
{
    const int lengths = blue64_classes();
    CHECK(lengths > 100);
    for (int nrings : {1, 2, 7, 8, 9, 15, 16, 17, 23, 24, 25, 31, 32, 33, 47, 48, 49})
        for (int nm : {1, 2, 5}) {
            for (int nmaps = 1; nmaps <= 17; ++nmaps) {
                one_to_one(sht::delta_blocked_maps(nm, nrings, nmaps), nmaps, nm, nrings);
                if (nmaps <= 3) {
                    one_to_one(sht::delta_blocked(nm, nrings), nmaps, nm, nrings);
                    one_to_one(sht::delta_plain(nm, nrings), nmaps, nm, nrings);
                }
            }
        }
    for (int count = 1; count <= 1100; count += count < 300 ? 1 : 37)
        for (int nitems : {1, 2, 3, 4, 8})
            for (int shift = 0; shift <= 4; ++shift) shares(count, nitems, shift);
    if (fail) return 1;
    std::printf("ring plan driver ok (%d convolution lengths)\n", lengths);
    return 0;
}
