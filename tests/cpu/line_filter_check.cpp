// Checks of the line filter's per-lane functions, compiled for the host.
// Usage: line_filter_check NAME; prints what fails and returns 1 if anything does.
#include "line_filter.h"

#include <barrier>
#include <cstdio>
#include <cstring>
#include <memory>
#include <random>
#include <thread>
#include <vector>

using namespace sphfilt;

static int failures = 0;
static std::unique_ptr<std::barrier<>> lanes;     // set while lanes run together

void lane_barrier()
{
    if (lanes) lanes->arrive_and_wait();
}

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

// Whole lines through the line filter, a thread per lane, sharp masks, against
// the circulant in long double: the largest error of a line relative to its
// largest value, averaged over random lines, is at most `most`.
template <int N, int LINES = 2000>
void line_error(double most)
{
    constexpr int N1 = Split<N>::N1, N2 = Split<N>::N2, NV = Split<N>::NV;
    const long double pi = 3.14159265358979323846264338327950288L;
    std::vector<Twiddle> table(N + N / 4);
    std::vector<long double> root(N);
    for (int j = 0; j < N; ++j) {
        const double c = (double)(root[j] = cosl(2 * pi * j / N)), s = (double)sinl(2 * pi * j / N);
        table[j] = Twiddle{c, -s};
        if (j < N / 4) table[N + j] = Twiddle{c, s / c};
    }
    std::mt19937_64 random(N);
    std::normal_distribution<double> normal;
    std::uniform_real_distribution<double> upto(0.0, 1.0);
    std::vector<std::vector<cplx>> x(LINES, std::vector<cplx>(N)), y = x;
    std::vector<double> cut(LINES);
    for (int i = 0; i < LINES; ++i) {
        cut[i] = 2.0 + upto(random) * (N / 2 - 2);
        for (cplx &z : x[i]) z = cplx{normal(random), normal(random)};
    }
    std::vector<double> lds(line_lds<N1, N2>());
    lanes = std::make_unique<std::barrier<>>(N2);
    std::vector<std::thread> threads;
    for (int t = 0; t < N2; ++t)
        threads.emplace_back([&, t] {
            for (int i = 0; i < LINES; ++i) {
                cplx v[NV] = {};
                for (int n = 0; n < N1; ++n) v[n] = x[i][N2 * n + t];
                filter_line<N1, N2, false, true>(v, t, 2, 2, false, cut[i], lds.data(), table.data());
                for (int n = 0; n < N1; ++n) y[i][N2 * n + t] = v[n];
                lane_barrier();
            }
        });
    for (std::thread &t : threads) t.join();
    lanes.reset();
    double sum = 0.0;
    for (int i = 0; i < LINES; ++i) {
        std::vector<long double> kernel(N, 0.0L);
        for (int d = 0; d < N; ++d)
            for (int q = 0; q < N; ++q)
                if ((q <= N / 2 ? q : N - q) <= cut[i]) kernel[d] += root[q * d % N] / N;
        long double size = 0.0L, error = 0.0L;
        for (int n = 0; n < N; ++n) {
            long double re = 0.0L, im = 0.0L;
            for (int k = 0; k < N; ++k) {
                re += kernel[(n - k + N) % N] * x[i][k].re;
                im += kernel[(n - k + N) % N] * x[i][k].im;
            }
            size = std::max(size, std::max(fabsl(re), fabsl(im)));
            error = std::max(error, std::max(fabsl(re - y[i][n].re), fabsl(im - y[i][n].im)));
        }
        sum += (double)(error / size);
    }
    if (!(sum / LINES <= most)) {
        std::printf("N %d: mean error %.4g, at most %.4g\n", N, sum / LINES, most);
        ++failures;
    }
}

#define EVERY_LENGTH(F)                                                                            \
    F<32>(), F<48>(), F<64>(), F<80>(), F<96>(), F<128>(), F<160>(), F<192>(), F<256>()

int main(int argc, char **argv)
{
    const char *name = argc > 1 ? argv[1] : "";
    if (!std::strcmp(name, "sharp")) EVERY_LENGTH(sharp);
    else if (!std::strcmp(name, "exponential")) EVERY_LENGTH(exponential);
    // the errors of the same transforms with all twiddles in full products on
    // both sides of the transposes, and 0.5 % for other compilers' contractions
    else if (!std::strcmp(name, "radix3_lines")) line_error<48>(1.005 * 2.883e-16), line_error<96>(1.005 * 3.016e-16);
    else if (!std::strcmp(name, "other_lines")) {
        line_error<32>(1.005 * 2.161e-16), line_error<64>(1.005 * 2.634e-16), line_error<80>(1.005 * 2.878e-16);
        line_error<128, 800>(1.005 * 2.915e-16), line_error<160, 600>(1.005 * 3.185e-16);
        line_error<256, 400>(1.005 * 3.163e-16);
    } else return 2;
    return failures ? 1 : 0;
}
