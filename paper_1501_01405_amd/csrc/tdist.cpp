// Student-t quantile for the replication confidence interval (the paper's
// section 1 interval from at least 30 replications; for fewer, the t law is
// the exact small-sample form of the same interval).
//
// Upper tail: P(T > t) = I_x(nu/2, 1/2) / 2 with x = nu / (nu + t^2), where
// I is the regularised incomplete beta function, evaluated by its continued
// fraction. The quantile starts from the normal one and the expansion of t
// in powers of 1 / nu, and is corrected by the inverse function's Taylor
// series to third order inside a bracket: one or two evaluations of the tail
// where an interval asks for it (0.35 us for 63 degrees of freedom and 0.975,
// where Newton from a bracket's middle took eight evaluations and 5.7 us).
// From ten thousand degrees of freedom on the expansion is the quantile.
#include <cmath>

namespace mrip {

namespace {

// log(Gamma(a + 1/2) / Gamma(a)). From 16 on by the ratio's asymptotic
// series (its first term left out is 2e-16 there); the difference of two
// logarithms loses as many digits as they are large.
double log_gamma_ratio(double a) {
  if (a < 16.0) return std::lgamma(a + 0.5) - std::lgamma(a);
  const double u = 1.0 / a, u2 = u * u;
  return 0.5 * std::log(a) +
         u * (-1.0 / 8 + u2 * (1.0 / 192 + u2 * (-1.0 / 640 + u2 * (17.0 / 14336 - u2 * (31.0 / 18432)))));
}

// Continued fraction for I_x(a, b), valid for x < (a + 1) / (a + b + 2): the
// convergents' numerators and denominators by their three-term recurrences,
// which keep divisions off the chain of dependent operations.
double beta_cf(double a, double b, double x) {
  const double eps = 1e-16;
  double p0 = 1.0, q0 = 1.0;  // convergent before the last
  double p1 = 1.0, q1 = 1.0 - (a + b) * x / (a + 1.0);
  for (int m = 1; m <= 10000; ++m) {
    const double m2 = 2.0 * m;
    const double even = m * (b - m) * x / ((a + m2 - 1.0) * (a + m2));
    const double odd = -(a + m) * (a + b + m) * x / ((a + m2) * (a + m2 + 1.0));
    const double p2 = p1 + even * p0, q2 = q1 + even * q0;
    const double p3 = p2 + odd * p1, q3 = q2 + odd * q1;
    const double cross = p3 * q1;  // p1 / q1 against p3 / q3
    if (std::fabs(cross - p1 * q3) <= eps * std::fabs(cross)) return p3 / q3;
    p0 = p2;
    q0 = q2;
    p1 = p3;
    q1 = q3;
    if (std::fabs(q1) < 1e-100) {
      p0 *= 1e100;
      q0 *= 1e100;
      p1 *= 1e100;
      q1 *= 1e100;
    } else if (std::fabs(q1) > 1e100) {
      p0 *= 1e-100;
      q0 *= 1e-100;
      p1 *= 1e-100;
      q1 *= 1e-100;
    }
  }
  return p1 / q1;
}

// Upper tail at t > 0, and the density there; `log_beta` is
// log B(nu / 2, 1 / 2).
double t_upper_tail(double t, double nu, double log_beta, double &pdf) {
  const double a = 0.5 * nu, r = t / nu * t;  // r = t^2 / nu
  const double x = 1.0 / (1.0 + r), y = r / (1.0 + r);
  // x^a y^(1/2) / B(a, 1/2)
  const double front = std::exp(-a * std::log1p(r) - log_beta) * std::sqrt(y);
  pdf = front / t;
  if (x < (a + 1.0) / (a + 2.5)) return 0.5 * front * beta_cf(a, 0.5, x) / a;
  return 0.5 - front * beta_cf(0.5, a, y);
}

// Standard normal quantile of an upper tail q < 1/2: a rational starting
// value (Abramowitz and Stegun 26.2.23, 4.5e-4) and third-order steps, of
// which one leaves some 1e-13 and two leave rounding.
double normal_upper(double q, int steps) {
  const double w = std::sqrt(-2.0 * std::log(q));
  double z = w - (2.515517 + w * (0.802853 + w * 0.010328)) /
                     (1.0 + w * (1.432788 + w * (0.189269 + w * 0.001308)));
  for (int i = 0; i < steps; ++i) {
    const double pdf = std::exp(-0.5 * z * z) * 0.3989422804014327;
    const double u = (0.5 * std::erfc(z * 0.7071067811865476) - q) / pdf;
    z += u * (1.0 + u * (0.5 * z + u * (2.0 * z * z + 1.0) / 6.0));
  }
  return z;
}

// The expansion of t in powers of 1 / nu (Abramowitz and Stegun 26.7.5) at the
// normal quantile z.
double t_expansion(double z, double nu) {
  const double z2 = z * z, v = 1.0 / nu;
  const double g1 = (z2 + 1.0) / 4, g2 = ((5.0 * z2 + 16.0) * z2 + 3.0) / 96;
  const double g3 = (((3.0 * z2 + 19.0) * z2 + 17.0) * z2 - 15.0) / 384;
  const double g4 = ((((79.0 * z2 + 776.0) * z2 + 1482.0) * z2 - 1920.0) * z2 - 945.0) / 92160;
  return z * (1.0 + v * (g1 + v * (g2 + v * (g3 + v * g4))));
}

}  // namespace

double t_quantile(double p, double nu) {
  if (!(p >= 0.5 && p < 1.0) || !(nu > 0.0)) return std::nan("");
  if (p == 0.5) return 0.0;
  const double target = 1.0 - p;  // upper-tail probability
  // From here on the expansion is exact to rounding (its next term is below
  // 1e-15 for any tail a double's p has), and the tail below is less and less
  // so: a log1p(r) of large a rounds to more than the steps' end asks for
  // (4.3e9 degrees of freedom: 62 us and an error of 1e-8 that way).
  if (nu >= 1e4) return t_expansion(normal_upper(target, 2), nu);
  const double log_beta = 0.5723649429247001 - log_gamma_ratio(0.5 * nu);  // log sqrt(pi) - ...
  double lo = 0.0, hi = INFINITY, pdf, t;
  if (nu >= 4.0 && target > 1e-12) {
    t = t_expansion(normal_upper(target, 1), nu);
  } else {
    double step = 1.0;
    while (t_upper_tail(step, nu, log_beta, pdf) > target) {
      lo = step;
      step *= 2.0;
      if (step > 1e300) return INFINITY;
    }
    hi = step;
    t = 0.5 * (lo + hi);
  }
  for (int it = 0; it < 200; ++it) {
    const double f = t_upper_tail(t, nu, log_beta, pdf) - target;  // decreasing in t
    if (f > 0) lo = t;
    else hi = t;
    // t as a function of the tail, from its derivatives: 1 / pdf, and with
    // c = -pdf' / pdf the higher ones
    const double u = f / pdf, s = nu + t * t;
    const double c = (nu + 1.0) * t / s, c1 = (nu + 1.0) * ((nu - t * t) / s) / s;
    const bool near = std::fabs(c * u) < 0.5;
    double next = near ? t + u * (1.0 + u * (0.5 * c + u * (2.0 * c * c + c1) / 6.0)) : t + u;
    // done when the fourth order would change nothing any more (asked before
    // the bracket, which rounding in f can have closed on t itself)
    const double k = 1.0 + c;
    if ((near && k * k * k * u * u * u * u <= 1e-17 * t) || std::fabs(next - t) <= 1e-15 * t)
      return next;
    if (!(next > lo && next < hi)) next = hi < INFINITY ? 0.5 * (lo + hi) : 2.0 * t;
    t = next;
    if (hi < INFINITY && hi - lo <= 1e-15 * hi) break;
  }
  return t;
}

}  // namespace mrip
