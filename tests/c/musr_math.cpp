// Host-only harness of csrc/musr_math.h: the quotient and the logarithm of the
// fit statistic against long double, with a reciprocal estimate of 22 bits.
// Prints, for each range of arguments, the largest and the root mean square
// error in units of the last place of the result.
//
//   g++ -std=c++17 -O2 -ffp-contract=off -I paper_1509_07685_amd/csrc tests/c/musr_math.cpp -o musr_math
#include "musr_math.h"

#include <cmath>
#include <cstdio>
#include <random>

static std::mt19937_64 gen(1);
static double uniform(double lo, double hi) { return lo + (hi - lo) * (double)(gen() >> 11) * 0x1p-53; }

struct Ops {
  static double estimate(double d) { return 1.0 / d * (1.0 + uniform(-0x1p-22, 0x1p-22)); }
  static double fma_const(double a, double b, double c) { return std::fma(a, b, c); }
};

static double ulps(double got, long double exact) {
  int e;
  frexpl(exact, &e);
  return (double)fabsl(((long double)got - exact) / ldexpl(1.0L, e - 53));
}

template <class F> static void report(const char* name, F&& f, int n) {
  double worst = 0.0, sum = 0.0;
  for (int i = 0; i < n; ++i) {
    const double u = f();
    worst = u > worst ? u : worst;
    sum += u * u;
  }
  std::printf("%s %.4f %.4f\n", name, worst, std::sqrt(sum / n));
}

int main() {
  using namespace dks::musr;
  auto log_err = [](double q) { return q == 1.0 ? 0.0 : ulps(log_normal<Ops>(q), logl((long double)q)); };
  auto div_err = [](double n, double d) { return ulps(quotient(n, d, recip<Ops>(d)), (long double)n / d); };
  const int n = 2000000;
  report("log_near_one", [&] { return log_err(1.0 + uniform(-0.01, 0.01)); }, n);
  report("log_ratio", [&] { return log_err(uniform(0.25, 4.0)); }, n);
  report("log_all", [&] { return log_err(std::ldexp(uniform(1.0, 2.0), (int)(gen() % 1919) - 959)); }, n);
  report("quotient_counts", [&] { return div_err(uniform(1e-3, 1e5), (double)(1 + gen() % 2000)); }, n);
  report("quotient_all", [&] { return div_err(std::ldexp(uniform(1.0, 2.0), (int)(gen() % 800) - 400),
                                              std::ldexp(uniform(1.0, 2.0), (int)(gen() % 800) - 400)); }, n);
  std::printf("log_one %.4f 0\n", std::fabs(log_normal<Ops>(1.0)));
  std::printf("zero_divisor %.4f 0\n", std::fabs(quotient(3.7, 0.0, 0.5) - 3.7));
  return 0;
}
