// The device's exponentials and quotients, compiled for the host, and libm's, against quad
// precision: largest and mean relative error of each, one line per function.
#include <cmath>
#include <cstdio>
#include <quadmath.h>
#include <random>
using std::isfinite;
#include "../../paper_2312_16981_amd/csrc/device_math.hpp"

typedef __float128 Q;
using namespace ugk;

template <class F, class G>
void measure(const char* name, F f, G exact, double lo, double hi)
{
    std::mt19937_64 gen(7);
    std::uniform_real_distribution<double> u(0.0, 1.0);
    const int n = 400000;
    double most = 0.0, sum = 0.0;
    for (int i = 0; i < n; ++i) {
        const double x = lo * std::pow(hi / lo, u(gen));
        const Q e = exact((Q)x);
        const double r = (double)fabsq(((Q)f(x) - e) / e);
        most = std::fmax(most, r);
        sum += r;
    }
    std::printf("%s %.6e %.6e\n", name, most, sum / n);
}

int main()
{
    const TabPtr t = math_tab();
    auto e = [](Q x) { return expq(-x); };
    auto o = [](Q x) { return -expm1q(-x); };
    measure("exp", [](double x) { return std::exp(-x); }, e, 1e-3, 700.0);
    measure("exp_neg_fine", [&](double x) { return exp_neg_fine(t, x); }, e, 1e-3, 700.0);
    measure("exp_neg", [&](double x) { return exp_neg(t, x); }, e, 1e-3, 700.0);
    measure("expm1", [](double x) { return -std::expm1(-x); }, o, 1e-6, 40.0);
    measure("one_less_exp_neg", [&](double x) { return one_less_exp_neg(t, x); }, o, 1e-6, 40.0);
    measure("sixth", [](double x) { return sixth(x); }, [](Q x) { return x / 6; }, 1e-6, 1e6);
    measure("over_pi4_15", [](double x) { return over_pi4_15(x); }, [](Q x) { return x / (Q)UGK_PI4_15; }, 1e-6, 1e6);
    const double ends[] = {0.0, 1e-300, 800.0, 1e300, INFINITY};
    for (double x : ends) std::printf("end %.17g %.17g %.17g\n", x, exp_neg_fine(t, x), one_less_exp_neg(t, x));
}
