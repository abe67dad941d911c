// track_check.cpp -- host check of the tracked images' last step (sblm_math.h,
// image_close): whatever start it is given, a point that it accepts solves the
// lens equation.  Prints per family of starts how many were tried and accepted,
// and the largest |residual|^2 / (1 + |z|^2) of an accepted point, in long
// double.  Families:
//   given     one start far out, beyond both lenses' reach
//   far       |z| from 10 to 10^150
//   random    anywhere near the lenses
//   critical  within 10^-6 ... 10^-15 of |g| = 1, from where a Newton step goes
//             anywhere
// and each goes through a Newton step (but `given` and `far`, which start at the
// judged one) and up to 8 judged ones, as a tracked epoch's images do.  Sources
// and lenses are drawn over the parameter domain, and one in four far outside.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>

namespace sblm {
static inline double fma(double a, double b, double c) { return std::fma(a, b, c); }
// (estimates as poor as the hardware's)
static inline double rcp_hw(double x) { return (1.0 / x) * (1.0 + 4e-8); }
static inline double rsq_hw(double x) { return (1.0 / std::sqrt(x)) * (1.0 - 4e-8); }
static inline double vmin(double a, double b) { return std::fmin(a, b); }
static inline double vmax(double a, double b) { return std::fmax(a, b); }
static inline double fabs(double a) { return std::fabs(a); }
using std::isfinite;
}  // namespace sblm

#include "sblm_math.h"

using sblm::cx;
typedef cx<double> C;

struct Lens {
  C zeta;
  double d, q;
};

// |residual|^2 / (1 + |z|^2) of the lens equation.
static double residual(C z, const Lens& l) {
  typedef long double L;
  const L x = z.re, y = z.im, ex = (L)l.d - x;
  const L n2 = x * x + y * y, e2 = ex * ex + y * y;
  const L re = l.zeta.re - x + x / n2 - (L)l.q * ex / e2;
  const L im = l.zeta.im - y + y / n2 + (L)l.q * y / e2;
  return (double)((re * re + im * im) / (1.0L + n2));
}

static std::mt19937_64 rng;
static double uni(double a, double b) {
  return a + (b - a) * ((double)(rng() >> 11) * 0x1p-53);
}

static Lens draw() {
  Lens l;
  const bool wide = (rng() & 3) == 0;
  l.q = std::pow(10.0, wide ? uni(-6, 2) : uni(-3, 0));
  l.d = wide ? std::pow(10.0, uni(-2.5, 1)) : uni(0.5, 2);
  const double r = wide ? std::pow(10.0, uni(-4, 2.3)) : uni(0, 3), a = uni(0, 2 * M_PI);
  l.zeta = {r * std::cos(a), r * std::sin(a)};
  return l;
}

struct Tally {
  long tried = 0, accepted = 0;
  double worst = 0.0;
  C z = {0, 0};
  Lens l = {{0, 0}, 0, 0};
};

static void judge(C z, const Lens& l, bool newton, Tally& t) {
  ++t.tried;
  if (newton) sblm::image_newton(z, l.zeta, l.d, l.q);
  for (int pass = 0; pass < 9; ++pass) {
    C g;
    double inv;
    if (!sblm::image_close(z, l.zeta, l.d, l.q, &g, &inv)) continue;
    ++t.accepted;
    const double r = residual(z, l);
    if (!(r <= t.worst)) t.worst = r, t.z = z, t.l = l;
    return;
  }
}

static void put(const char* name, const Tally& t, const char* end) {
  std::printf("\"%s\": {\"tried\": %ld, \"accepted\": %ld, \"worst\": %.3e, \"zeta\": [%.17g, "
              "%.17g], \"d\": %.17g, \"q\": %.17g}%s\n",
              name, t.tried, t.accepted, std::isfinite(t.worst) ? t.worst : 1e300, t.l.zeta.re,
              t.l.zeta.im, t.l.d, t.l.q, end);
}

int main(int argc, char** argv) {
  const long n = argc > 1 ? std::atol(argv[1]) : 1000000;
  rng.seed(argc > 2 ? std::strtoull(argv[2], nullptr, 10) : 1);
  Tally given, far, random, critical;
  judge({2e6, 6e5}, {{-0.1457, 0.1939}, 1.9607, 0.002876}, false, given);
  for (long k = 0; k < n; ++k) {
    const Lens l = draw();
    const double a = uni(0, 2 * M_PI);
    {
      const double r = std::pow(10.0, (k & 1) ? uni(1, 12) : uni(12, 150));
      judge({r * std::cos(a), r * std::sin(a)}, l, false, far);
    }
    const double r = std::pow(10.0, uni(-3, 0.6)), c = (k & 1) ? l.d : 0.0;
    judge({c + r * std::cos(a), r * std::sin(a)}, l, true, random);
    // |g| falls from 1/r^2 at a lens to 0 far out: bisect for |g| = 1 along a ray
    auto excess = [&](double s) {
      return sblm::c_norm(sblm::lens_at<true>(C{c + s * std::cos(a), s * std::sin(a)}, l.zeta,
                                              l.d, l.q).g) - 1.0;
    };
    double lo = 1e-6, hi = 1e3;
    if (!(excess(lo) > 0.0 && excess(hi) < 0.0)) continue;
    for (int b = 0; b < 90 && hi - lo > 1e-16 * hi; ++b) {
      const double m = 0.5 * (lo + hi);
      if (m == lo || m == hi) break;
      (excess(m) > 0.0 ? lo : hi) = m;
    }
    const double s = lo * (1.0 + std::pow(10.0, uni(-15.5, -6)) * ((rng() & 1) ? 1.0 : -1.0));
    judge({c + s * std::cos(a), s * std::sin(a)}, l, true, critical);
  }
  std::printf("{");
  put("given", given, ",");
  put("far", far, ",");
  put("random", random, ",");
  put("critical", critical, "}");
  return 0;
}
