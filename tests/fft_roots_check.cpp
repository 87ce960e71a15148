// The roots of unity of the transforms in fft_regs.h, evaluated on the host and compared with long double: angles, tables,
// products. Built and run by tests/test_fft_roots.py; prints the largest errors and exits 0 when every bound holds.
#include <cmath>
#include <cstdio>
#include <vector>

#include "fft_regs.h"

using namespace audiokv;

static int failed = 0;
// largest error of a float32 root over both parts: half an ulp of [1/2, 1) when rounded once
static const double kOnce = std::ldexp(1.0, -25) + 1e-11;

struct Worst {
    const char* name;
    double bound, err = 0;
    void add(cf w, long double x) {                       // w against exp(i pi x)
        const long double a = 3.14159265358979323846264338327950288L * x;
        err = std::fmax(err, std::fmax(std::fabs((double)(w.re - std::cos(a))), std::fabs((double)(w.im - std::sin(a)))));
    }
    ~Worst() {
        std::printf("%-28s %.3e (bound %.3e)\n", name, err, bound);
        if (!(err <= bound)) ++failed;
    }
};

template <int LOGC>
void table_of_roots() {
    using F = Fft<LOGC, 1, true>;
    std::vector<cf> table(padded_len(F::C / 2));
    for (int t = 0; t < F::THREADS; ++t) F::fill_table(table.data(), t);
    Worst roots{"table", kOnce}, bins{"bins", kOnce};
    for (int e = 0; e < F::C / 2; ++e) roots.add(table[pad(e)], -(long double)e / (F::C / 2));
    for (int t = 0; t < F::THREADS; ++t) {
        typename F::Twiddles tw;
        F::init(tw, table.data(), t);
        for (int p = 0; p < F::TW; ++p) {
            const cf w[8] = {{1.f, 0.f}, tw.w[0][p].w1, tw.w[0][p].w2, tw.w[0][p].w3, tw.w[0][p].w4, tw.w[0][p].w5, tw.w[0][p].w6, tw.w[0][p].w7};
            for (int k = 0; k < 8; ++k) roots.add(w[k], -(long double)(k * F::exponent(p, t)) / (F::C / 2));
        }
        const typename F::BinRoots root(t);
        for (int e = 0; e < 8; ++e) bins.add(root(e), -(long double)F::bin_of(8 * t + e) / F::C);
    }
}

int main() {
    {
        Worst any{"angles", kOnce};
        for (int k = -(1 << 18); k <= (1 << 18); ++k) any.add(cis_pi((float)k / 65536.f), (long double)k / 65536);
        for (int n = 1; n < 2000; ++n) for (int k = 0; k <= n; k += 1 + n / 50) { const float x = (float)k / (float)n; any.add(cis_pi(x), x); }
    }
    table_of_roots<9>();
    table_of_roots<10>();
    table_of_roots<11>();
    table_of_roots<12>();
    table_of_roots<13>();
    {
        // 16384 points: every fourth root in the table, the others within the rounding of their neighbour and their own
        using F = Fft<14, 2>;
        std::vector<cf> table(padded_len(F::C / 8));
        for (int t = 0; t < F::THREADS; ++t) F::fill_every_fourth(table.data(), t);
        Worst between{"between table entries", 2 * kOnce}, entries{"table of every fourth", kOnce}, bins{"bins", kOnce};
        for (int t = 0; t < F::THREADS; ++t) {
            const typename F::EveryFourth tw(table.data(), t);
            for (int vt = 0; vt < 2; ++vt) {
                for (int p = 0; p < F::TW; ++p) {
                    const int e = F::exponent(p, t + vt * F::THREADS);
                    const typename F::W3 w = tw(p, vt);
                    (p ? entries : between).add(w.w1, -(long double)e / (F::C / 2));
                    (p ? entries : between).add(w.w2, -(long double)(2 * e) / (F::C / 2));
                    entries.add(w.w4, -(long double)(4 * e) / (F::C / 2));
                }
                const typename F::BinRoots root(t + vt * F::THREADS);
                for (int e = 0; e < 8; ++e) bins.add(root(e), -(long double)F::bin_of(8 * (t + vt * F::THREADS) + e) / F::C);
            }
        }
    }
    std::printf(failed ? "%d bounds exceeded\n" : "all bounds hold\n", failed);
    return failed != 0;
}
