// Checks of the line filter's per-lane functions, compiled for the host.
// Usage: line_filter_check NAME; prints what fails and returns 1 if anything does.
#include "line_filter.h"

#include <cstdio>
#include <cstring>
#include <random>

using namespace sphfilt;

static int failures = 0;

template <int N, typename Apply>
void mask_of(double (&f)[N], Apply &&apply)
{
    constexpr int N1 = Split<N>::N1, N2 = Split<N>::N2, NV = Split<N>::NV;
    for (int t = 0; t < N2; ++t) {
        cplx v[NV];
        for (cplx &x : v) x = cplx{1.0, 1.0};
        apply(v, t);
        for (int r = 0; r < NV / N2; ++r)
            for (int k2 = 0; k2 < N2; ++k2)
                if (t + N2 * r < N1) f[t + N2 * r + N1 * k2] = v[r * N2 + k2].re;
    }
}

static double ulps_from(double x, int k)
{
    for (; k > 0; --k) x = std::nextafter(x, INFINITY);
    for (; k < 0; ++k) x = std::nextafter(x, -INFINITY);
    return x;
}

// A sharp mask keeps a mode exactly when |q| <= c, also where c lies a few
// units of its last place from an integer.
template <int N>
void sharp()
{
    constexpr int N1 = Split<N>::N1, N2 = Split<N>::N2;
    double f[N];
    auto check = [&](double c, const char *form) {
        for (int q = 0; q < N; ++q) {
            const int a = q <= N / 2 ? q : N - q;
            if (f[q] == ((double)a <= c ? 1.0 / N : 0.0)) continue;
            std::printf("N %d %s: mode %d at cutoff %.17g has factor %g / N\n", N, form, q, c, f[q] * N);
            ++failures;
        }
    };
    for (int m = 0; m <= N / 2; ++m)
        for (int k = -3; k <= 3; ++k) {
            const double c = ulps_from(m, k);
            if (c < 0.0) continue;
            mask_of<N>(f, [&](auto &v, int t) { apply_mask<N1, N2>(v, t, 2, c); });
            check(c, "apply_mask");
            mask_of<N>(f, [&](auto &v, int t) { apply_mask_two<N1, N2>(v, t, true, c); });
            check(c, "apply_mask_two");
        }
}

// The exponential factors are min(1, e^{c - |q|}) / N to the roundings that they
// are formed by: the exponential's argument (relative to its size) and value,
// two constants that are rounded and multiply it, and, where N is not a power of
// two, 1 / N, its product and the check's own.
template <int N>
void exponential()
{
    constexpr int N1 = Split<N>::N1, N2 = Split<N>::N2;
    constexpr double u = 0x1p-53;
    constexpr double fixed = ((N & (N - 1)) == 0 ? 5.1 : 8.1) * u;
    double f[N];
    auto check = [&](double c, const char *form) {
        for (int q = 0; q < N; ++q) {
            const int a = q <= N / 2 ? q : N - q;
            const long double want = a <= c ? 1.0L : expl((long double)c - a);
            const double err = (double)(fabsl((long double)f[q] * N - want) / want);
            if (err <= fixed + u * (a > c ? a - c : 0.0)) continue;
            std::printf("N %d %s: mode %d at cutoff %.17g: relative error %.3g\n", N, form, q, c, err);
            ++failures;
        }
    };
    std::mt19937_64 random(N);
    std::uniform_real_distribution<double> upto(0.0, 1.0);
    for (int i = 0; i < 4000; ++i) {
        const double c = i % 2 ? upto(random) * N / 2 : i % 4 ? upto(random) * 20.0 : (double)(i / 4 % (N / 2));
        mask_of<N>(f, [&](auto &v, int t) { apply_mask<N1, N2>(v, t, 0, c); });
        check(c, "apply_mask");
        mask_of<N>(f, [&](auto &v, int t) { apply_mask_two<N1, N2>(v, t, false, c); });
        check(c, "apply_mask_two");
        // the two-kind mask with one kind for both lines: with two the factor
        // itself cannot be read from the sum of halves that it applies
        double other[N];
        for (double &x : other) x = 1.0;
        mask_of<N>(f, [&](auto &v, int t) { apply_mask_pair<N1, N2, true>(v, t, 0, 0, c, other); });
        check(c, "apply_mask_pair");
    }
    // cutoffs above every mode, up to infinity
    for (double c : {0.5 * N, 1.0 * N, 700.0, 712.5, 1e300, (double)INFINITY}) {
        mask_of<N>(f, [&](auto &v, int t) { apply_mask<N1, N2>(v, t, 0, c); });
        check(c, "apply_mask");
        mask_of<N>(f, [&](auto &v, int t) { apply_mask_two<N1, N2>(v, t, false, c); });
        check(c, "apply_mask_two");
    }
}

#define EVERY_LENGTH(F)                                                                            \
    F<32>(), F<48>(), F<64>(), F<80>(), F<96>(), F<128>(), F<160>(), F<192>(), F<256>()

int main(int argc, char **argv)
{
    const char *name = argc > 1 ? argv[1] : "";
    if (!std::strcmp(name, "sharp")) EVERY_LENGTH(sharp);
    else if (!std::strcmp(name, "exponential")) EVERY_LENGTH(exponential);
    else return 2;
    return failures ? 1 : 0;
}
