// Host harness for the device's form of the FP64 log and exp of the sampling path: the
// library's own header, built with the host compiler and -ffp-contract=off, with the
// hardware reciprocal replaced by an estimate whose relative error is anywhere within
// +-2^-23.  Prints the quotient's largest distance from the exact one in units of the last
// place (half a unit is a correct rounding), the largest errors of log_pos and exp_core
// against the x87 extended-precision logl / expl as in math_f64_check.cpp, then "ok" or the
// first failing special value (exit status 1).
#include <algorithm>
#include <cfloat>
#include <cmath>
#include <cstdint>
#include <cstdio>

namespace {

uint64_t rs = 0x9E3779B97F4A7C15ull;
double uniform() {  // [0, 1)
  rs ^= rs << 13;
  rs ^= rs >> 7;
  rs ^= rs << 17;
  return double(rs >> 11) * 0x1p-53;
}

// an estimate of 1 / d: at either end of the error range half of the time
double seed(double d) {
  const double u = uniform();
  const double e = u < 0.25 ? -1.0 : u < 0.5 ? 1.0 : 2.0 * uniform() - 1.0;
  return (1.0 / d) * (1.0 + e * 0x1p-23);
}

}  // namespace

#define R1X_RCP_SEED seed
#include "r1_math.hpp"

namespace {

double ulps(double got, long double ref) {
  int e;
  std::frexp(double(ref), &e);
  return double(std::fabs((long double)got - ref)) / std::ldexp(1.0, std::max(e - 53, -1074));
}

template <typename F, typename G, typename R>
void max_ulp(const char* name, int n, G gen, F f, R ref) {
  double worst = 0.0, at = 0.0;
  for (int i = 0; i < n; ++i) {
    const double x = gen();
    const double u = ulps(f(x), ref(x));
    if (!(u <= worst)) { worst = u; at = x; }
  }
  std::printf("max_ulp %s %.6f at %.17g\n", name, worst, at);
}

}  // namespace

int main() {
  const int n = 2000000;
  // the reduction's operands: f = m - 1, m in [sqrt(1/2), sqrt(2)), over 2 + f, down to tiny f
  auto quotient = [](double f) { return r1x::near_one_quotient(f, 2.0 + f); };
  auto quotient_l = [](double f) { return (long double)f / (long double)(2.0 + f); };
  max_ulp("quotient", n, [] { return 0.7071067811865476 + 0.7071067811865475 * uniform() - 1.0; }, quotient, quotient_l);
  max_ulp("quotient_small", n, [] { return std::ldexp(uniform() < 0.5 ? -1.0 - uniform() : 1.0 + uniform(), -2 - int(uniform() * 51)); },
          quotient, quotient_l);
  auto lg = [](double x) { return r1x::log_pos(x); };
  auto lgr = [](double x) { return logl((long double)x); };
  auto ex = [](double v) { return r1x::exp_core(v); };
  auto exr = [](double v) { return expl((long double)v); };
  max_ulp("log_all", n, [] { return std::ldexp(1.0 + uniform(), int(uniform() * 2097) - 1074); }, lg, lgr);
  max_ulp("log_near1", n, [] { return 0.5 + 1.5 * uniform(); }, lg, lgr);
  max_ulp("log_1pm", n, [] { return 1.0 + (uniform() - 0.5) * 1e-6; }, lg, lgr);
  max_ulp("exp_neg", n, [] { return -745.0 * uniform(); }, ex, exr);
  max_ulp("exp_unit", n, [] { return -uniform(); }, ex, exr);
  max_ulp("exp_pos", n, [] { return 700.0 * uniform(); }, ex, exr);
  const bool special = r1x::log_pos(1.0) == 0.0 && std::isnan(r1x::log_pos(0.0)) && std::isnan(r1x::log_pos(-1.0)) &&
                       std::isnan(r1x::log_pos(HUGE_VAL)) && std::isnan(r1x::log_pos(NAN)) &&
                       r1x::exp_core(0.0) == 1.0 && r1x::exp_core(-746.0) == 0.0 && std::isnan(r1x::exp_core(NAN));
  std::printf(special ? "ok\n" : "special\n");
  return special ? 0 : 1;
}
