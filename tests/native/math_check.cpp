// Errors of the exponentials and logarithms of bn_math.h (host form) against
// long double (64-bit significand), in units of the last place, over the ranges
// that the lattice kernels use and around the points where the functions change
// form. The bounds are the largest errors of the device library's exp, log and
// log1p over the same ranges.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <random>

#include "../../paper_1408_1664_amd/csrc/bn_math.h"

static constexpr int kCount = 1 << 19;
static int failed = 0;

static double ulps(double got, long double want) {
    if (want == 0.0L) return got == 0.0 ? 0.0 : HUGE_VAL;
    int e;
    std::frexp(want, &e);
    return (double)(fabsl((long double)got - want) / std::ldexp(1.0L, std::max(e, -1021) - 53));
}

template <class F, class T, class G>
static void check(const char *name, double bound, F f, T truth, G arg) {
    std::mt19937_64 gen(3);
    std::uniform_real_distribution<double> unit(0.0, 1.0);
    double worst = 0.0, at = 0.0;
    for (int i = 0; i < kCount; ++i) {
        const double x = arg(unit(gen), i);
        const double u = ulps(f(x), truth(x));
        if (!(u <= worst)) worst = u, at = x;
    }
    const bool ok = worst <= bound;
    failed += ok ? 0 : 1;
    printf("%s %s: %.4f ulp at %.17g (bound %.2f)\n", ok ? "ok  " : "FAIL", name, worst, at, bound);
}

static void expect(const char *name, bool ok) {
    failed += ok ? 0 : 1;
    printf("%s %s\n", ok ? "ok  " : "FAIL", name);
}

// the i-th double from x0
static double step(double x0, int i) {
    double x = x0;
    for (int k = 0; k < (i & 63); ++k) x = std::nextafter(x, i & 64 ? 10.0 : -10.0);
    return x;
}

int main() {
    using namespace bnk;
    constexpr double kExp = 0.88, kLog = 0.64;
    auto e0 = [](double x) { return exp_scaled(x, 0); };
    auto te = [](double x) { return expl(x); };
    check("exp, [-1, 0]", kExp, e0, te, [](double u, int) { return -u; });
    check("exp, [-40, 0]", kExp, e0, te, [](double u, int) { return -40.0 * u; });
    check("exp, [-700, 700]", kExp, e0, te, [](double u, int) { return 1400.0 * u - 700.0; });
    check("exp, near the edges of the reduction", kExp, e0, te, [](double u, int i) {
        return ((i % 401) - 200 + 0.5) * 0.69314718055994531 * (1.0 + (u - 0.5) * 1e-6);
    });
    check("exp, small", kExp, e0, te, [](double u, int) { return -std::exp2(-80.0 * u); });
    check("exp 2^960, [-1200, 0]", kExp, [](double x) { return exp_scaled(x, 960); },
          [](double x) { return std::ldexp(expl(x), 960); }, [](double u, int) { return -1200.0 * u; });
    check("exp 2^-1000, [0, 1300]", kExp, [](double x) { return exp_scaled(x, -1000); },
          [](double x) { return std::ldexp(expl(x), -1000); }, [](double u, int) { return 1300.0 * u; });
    auto l0 = [](double y) { return log_pos(y); };
    auto tl = [](double y) { return logl(y); };
    check("log, [1/2, 2]", kLog, l0, tl, [](double u, int) { return 0.5 + 1.5 * u; });
    check("log, 1 + 2^-50 .. 2", kLog, l0, tl, [](double u, int) { return 1.0 + std::exp2(-50.0 * u); });
    check("log, 1 - 2^-50 .. 1/2", kLog, l0, tl, [](double u, int) { return 1.0 - 0.5 * std::exp2(-50.0 * u); });
    check("log, [1, 31]", kLog, l0, tl, [](double u, int) { return 1.0 + 30.0 * u; });
    check("log, 2^-1000 .. 2^1000", kLog, l0, tl, [](double u, int) { return std::exp2(2000.0 * u - 1000.0); });
    check("log, subnormal", kLog, l0, tl, [](double u, int) { return std::ldexp(0.5 + 0.5 * u, -1030); });
    check("log, where the form changes", kLog, l0, tl,
          [](double, int i) { return step(std::ldexp(0.70710678118654757, i % 40 - 20), i); });
    check("log(y 2^1000), y about 2^-1000", kLog, [](double y) { return log_scaled(y, -1000); },
          [](double y) { return logl(std::ldexp((long double)y, 1000)); },
          [](double u, int) { return std::ldexp(1.0 + std::exp2(-50.0 * u), -1000); });
    auto p0 = [](double x) { return log1p_unit(x); };
    auto tp = [](double x) { return log1pl(x); };
    check("log1p, [0, 1]", kLog, p0, tp, [](double u, int) { return u; });
    check("log1p, 2^-1000 .. 1", kLog, p0, tp, [](double u, int) { return std::exp2(-1000.0 * u); });
    check("log1p, where the form changes", kLog, p0, tp,
          [](double, int i) { return step(i & 128 ? 0.41421356237309503 : 0.5, i); });
    expect("exp(-inf) = 0", exp_scaled(-HUGE_VAL, 960) == 0.0 && exp_neg(-HUGE_VAL) == 0.0);
    expect("exp of NaN is no NaN", exp_neg(NAN) == 0.0);
    expect("exp overflows to inf", exp_scaled(1500.0, -1000) == HUGE_VAL && exp_scaled(1e9, 0) == HUGE_VAL);
    expect("exp(0) = 1, log(1) = 0, log1p(0) = 0",
           exp_neg(0.0) == 1.0 && log_pos(1.0) == 0.0 && log1p_unit(0.0) == 0.0);
    expect("log(2^k 2^-k) = 0", log_scaled(0x1p960, 960) == 0.0 && log_scaled(0x1p-1000, -1000) == 0.0);
    // a million terms of e^-37 added to 1 one by one, as logarithms
    double acc = 0.0;
    for (int i = 0; i < 1000000; ++i) {
        const double t = -37.0;
        const double hi = std::max(acc, t), lo = std::min(acc, t);
        acc = hi + log1p_unit(exp_neg(lo - hi));
    }
    expect("small terms add up", std::fabs(acc / log1p(1e6 * exp(-37.0)) - 1.0) < 1e-9);
    return failed ? 1 : 0;
}
