// The register-local u32 networks of bcf_device.hpp, run on the host.  They
// consist of minima and maxima only, so by the 0-1 principle the 0-1 inputs
// decide them; every 0-1 input of each network's precondition is tried.
#include <stdint.h>
#include <stdio.h>

#include "bcf_device.hpp"

using namespace bcf;

namespace {

int g_bad = 0;

void expect_sorted(const Lines<false> &t, int lo, int n, bool desc, const char *what, int a, int b)
{
    for (int i = lo; i + 1 < lo + n; ++i)
        if (desc ? t.k[i] < t.k[i + 1] : t.k[i] > t.k[i + 1]) {
            if (g_bad++ < 5)
                printf("%s: input (%d, %d) of %d keys not sorted at %d\n", what, a, b, n, i);
            return;
        }
}

// Two sorted halves with a and b ones.
template <int LO, int N>
void merges()
{
    for (int a = 0; a <= N / 2; ++a)
        for (int b = 0; b <= N / 2; ++b) {
            Lines<false> t{};
            for (int i = 0; i < N / 2; ++i) {
                t.k[LO + i] = i >= N / 2 - a;
                t.k[LO + N / 2 + i] = i >= N / 2 - b;
            }
            oe_merge_keys<LO, N>(t);
            expect_sorted(t, LO, N, false, "oe_merge_keys", a, b);
        }
}

// Every cyclic 0-1 bitonic sequence in every aligned group of 2D registers.
template <int D, int DB>
void cleans()
{
    const int n = 2 * D;
    for (int ones = 0; ones <= n; ++ones)
        for (int at = 0; at < n; ++at) {
            Lines<false> t{};
            for (int r = 0; r < kLine; ++r)
                t.k[r] = (r % n + n - at) % n < ones;
            half_clean_lines<D, DB>(t);
            for (int g = 0; g < kLine; g += n)
                expect_sorted(t, g, n, DB >= 0 && ((g >> (DB < 0 ? 0 : DB)) & 1), "half_clean_lines", ones, at);
        }
}

template <int D>
void cleans_all()
{
    cleans<D, -1>();
    if constexpr (2 * D < kLine)
        cleans<D, log2i(2 * D)>();
    if constexpr (D > 1)
        cleans_all<D / 2>();
}

}  // namespace

int main()
{
    for (int m = 0; m < 16; ++m) {
        Lines<false> t{};
        for (int i = 0; i < 4; ++i)
            t.k[i] = (m >> i) & 1;
        sort4<0>(t);
        expect_sorted(t, 0, 4, false, "sort4", m, 0);
    }
    merges<0, 8>();
    merges<8, 8>();
    merges<16, 16>();
    merges<32, 32>();
    merges<0, 64>();
    cleans_all<kLine / 2>();
    // the line sort: keys of every width, the multiset kept
    uint64_t x = 1;
    for (int it = 0; it < 20000; ++it) {
        Lines<false> t;
        uint32_t in[kLine];
        for (int r = 0; r < kLine; ++r) {
            x = x * 6364136223846793005ull + 1442695040888963407ull;
            t.k[r] = in[r] = (uint32_t)(x >> 32) >> (it % 32);
        }
        oe_sort_lines<0, kLine - 1>(t);
        expect_sorted(t, 0, kLine, false, "oe_sort_lines", it, 0);
        for (int r = 0; r < kLine; ++r) {
            int had = 0, has = 0;
            for (int q = 0; q < kLine; ++q) {
                had += in[q] == in[r];
                has += t.k[q] == in[r];
            }
            if (had != has && g_bad++ < 5)
                printf("oe_sort_lines: input %d: key %u %d times, was %d\n", it, in[r], has, had);
        }
    }
    printf("%d failures\n", g_bad);
    return g_bad ? 1 : 0;
}
