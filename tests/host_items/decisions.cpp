// Host check of the decisions that the kernels take without the logarithm,
// exponential or quotient they are defined by (srk_device.hpp,
// flash_stages.hpp): each shortcut against the definition on random inputs
// and on inputs next to the threshold.  Prints one line per decision:
// name, cases, contradictions, cases the shortcut settled.
#include <cstdint>
#include <cstdio>
#include <random>

#include "flash_stages.hpp"

using namespace ptf;

static std::mt19937_64 rng(12345);
static double uni(double a, double b) { return std::uniform_real_distribution<double>(a, b)(rng); }
static double lg(double a, double b) { return std::exp(uni(std::log(a), std::log(b))); }

static double gibbs(double A, double B, double z)
{
    return z - 1.0 - log(z - B) - (A / B) * log1p(B / z);
}

int main()
{
    // Gibbs order of two roots: zl, zv over the whole range, and pairs whose
    // energies nearly tie (A solved from gv = gl, then moved by a relative d)
    long n = 0, bad = 0, set = 0;
    for (long k = 0; k < 4000000; ++k) {
        const double B = lg(1e-12, 0.5);
        const double zl = B * (1.0 + lg(1e-6, 10.0));
        const double zv = zl * (1.0 + lg(1e-9, 1e3));
        if (!(zv < 1.0 + B)) continue;
        const double num = (zv - zl) - (log(zv - B) - log(zl - B));
        const double den = (log1p(B / zv) - log1p(B / zl)) / B;
        double A = k % 2 ? lg(1e-10, 30.0) : num / den;
        if (k % 2 == 0) A *= 1.0 + (uni(-1, 1) < 0 ? -1 : 1) * lg(1e-14, 1e-1);
        if (!(A > 0.0) || !std::isfinite(A)) continue;
        const int s = gibbs_order(A, B, zl, zv);
        const double gl = gibbs(A, B, zl), gv = gibbs(A, B, zv);
        ++n;
        set += s != 0;
        bad += (s < 0 && !(gv < gl)) || (s > 0 && gv < gl);
    }
    // values single precision cannot hold, and equal roots, are left open
    bad += gibbs_order(1e-40, 1e-41, 2e-41, 1.0) != 0;
    bad += gibbs_order(0.3, 0.05, 0.2, 0.2) != 0;
    bad += gibbs_order(NAN, 0.05, 0.2, 0.3) != 0;
    bad += gibbs_order(INFINITY, 0.05, 0.2, 0.3) != 0;
    printf("gibbs_order %ld %ld %ld\n", n, bad, set);

    // substitution convergence
    n = bad = set = 0;
    const double tols[] = {1e-18, 1e-16, 1e-12, 1e-8, 1e-3, 0.05, 0.5, 2.0};
    for (long k = 0; k < 800000; ++k) {
        const double tol = tols[k % 8];
        double s[3], smax = 0.0;
        for (int i = 0; i < 3; ++i) {
            s[i] = (k % 3 == 0 ? uni(-3, 3) : tol * lg(1e-2, 1e2)) * (uni(-1, 1) < 0 ? -1 : 1);
            if (k % 1000 == 7 && i == 1) s[i] = k % 2000 == 7 ? INFINITY : NAN;
            smax = fmax(smax, fabs(s[i]));
        }
        const bool near = smax <= ss_far(tol);
        ++n;
        set += !near;
        bad += !near && ss_converged<3>(s, tol);
    }
    printf("ss_far %ld %ld %ld\n", n, bad, set);

    // trivial split
    n = bad = set = 0;
    for (long k = 0; k < 800000; ++k) {
        double x[3], y[3], lk = 0.0;
        for (int i = 0; i < 3; ++i) {
            x[i] = lg(1e-12, 1.0);
            y[i] = x[i] * (1.0 + (k % 2 ? lg(1e-9, 1e-4) : lg(1e-7, 5e-6)) * (uni(-1, 1) < 0 ? -1 : 1));
            if (k % 500 == 3 && i == 2) x[i] = 0.0;
            if (k % 500 == 4 && i == 2) y[i] = 0.0;
            if (k % 500 == 5 && i == 2) x[i] = -x[i];
            if (k % 500 == 6 && i == 2) y[i] = -y[i];
            if (k % 500 == 8 && i == 2) x[i] = NAN;
            lk = fmax(lk, fabs(log(y[i] / x[i])));
        }
        ++n;
        set += lk < 1e-6;
        bad += trivial_split<3>(x, y) != (lk < 1e-6);
    }
    printf("trivial_split %ld %ld %ld\n", n, bad, set);

    // step cut
    n = bad = set = 0;
    for (long k = 0; k < 800000; ++k) {
        const double v = k % 50 == 9 ? 0.0 : lg(1e-15, 1.0), z = v + (k % 40 == 9 ? 0.0 : lg(1e-15, 1.0));
        double u = v * lg(1e-3, 1e3) * (uni(-1, 1) < 0 ? -1 : 1);
        if (k % 60 == 1) u = 0.99 * v;
        if (k % 60 == 2) u = -0.99 * v;
        if (k % 60 == 3) u = 0.0;
        if (k % 60 == 4) u = NAN;
        if (k % 60 == 5) u = INFINITY;
        const double a0 = k % 2 ? 1.0 : uni(0, 1);
        double want = a0;
        if (u < 0.0) want = fmin(want, 0.99 * v / -u);
        if (u > 0.0) want = fmin(want, 0.99 * (z - v) / u);
        const double got = cut_step(a0, u < 0.0 ? v : z - v, fabs(u));
        ++n;
        set += got < a0;
        bad += !(got == want);
    }
    printf("cut_step %ld %ld %ld\n", n, bad, set);
    return 0;
}
