// Host tables of libvie: quadrature rules, special functions and the per-fill
// Ewald lattice-sum tables (Sec. 2.2, Eqs. 3-4 and the Ewald split).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <atomic>
#include <system_error>
#include <thread>
#include <vector>

#include "host.h"

namespace vie {

static const double kPi = 3.14159265358979323846;

using ld = long double;

// ---------------------------------------------------------------- special functions
// The Ewald terms are integrals over the split variable (in units of E) with
// a real wavenumber, so their expansion in the wavenumber,
//   int_1^inf s^(-2 first) exp(-x^2 s^2 + c / s^2) ds = sum_n c^n / n! J_{n+first}(x),
//   J_n(x) = int_1^inf s^(-2n) exp(-x^2 s^2) ds,
// has terms of one sign for c >= 0 and needs nothing but erfc: J_1 = e^{-x^2}
// - sqrt(pi) x erfc(x) and, by parts, J_{n+1} = (e^{-x^2} - 2 x^2 J_n) /
// (2n + 1).  The recurrence loses at most a factor e^{x^2} of terms of size
// e^{-x^2}, so a sum is good to some 1e-19 absolute (extended precision),
// where the fits resolve 1e-15.  This is a few dozen operations per value:
// quadrature of the complex erfcx integrals took 60 ms of host time per fill
// (16-18 ms on 16 threads), the tables now take 2 ms on one.  The far entries of
// the mixed operator keep to the quadratures below (PgfTerms::fixed).
// Sum over n >= n0 of c^n / n! J_{n + first}(x), n0 + first >= 1.
static const ld kSqrtPiL = 1.772453850905516027298167483341145183L;

static ld tail_sum(ld x, ld c, int first, int n0) {
  const ld e = std::exp(-x * x), x2 = 2 * x * x;
  ld J = e - kSqrtPiL * x * std::erfc(x);   // J_1
  for (int k = 1; k < n0 + first; ++k) J = (e - x2 * J) / (2 * k + 1);
  ld coef = 1, sum = 0;
  for (int n = 1; n <= n0; ++n) coef *= c / n;
  for (int n = n0; n < 400; ++n) {
    const ld term = coef * J;
    sum += term;
    if (n > c && term < 1e-22L * sum) break;
    J = (e - x2 * J) / (2 * (n + first) + 1);
    coef *= c / (n + 1);
  }
  return sum;
}

// The same functions by Gauss-Legendre quadrature of erfcx(z) = (2 / sqrt(pi))
// int_0^inf exp(-s^2 - 2 z s) ds (Re z >= 0; composite, up to where the
// integrand falls below 1e-20) and erf(z) = (2 z / sqrt(pi)) int_0^1
// exp(-z^2 t^2) dt, in extended precision.  The mixed-precision operator takes
// its terms from these (PgfTerms::fixed): both evaluations are good to some
// 1e-19, and so differ in the last bit of one coefficient in a few hundred,
// which is enough to move isolated FP32 entries of Z to their neighbours.
using zl = std::complex<long double>;

// Nodes and weights on [0, 1] by Newton iteration on the Legendre three-term
// recurrence.
static void gauss_legendre01(int n, std::vector<ld> &x, std::vector<ld> &w) {
  x.resize(n);
  w.resize(n);
  const ld pi = 3.141592653589793238462643383279502884L;
  for (int i = 0; i < n; ++i) {
    ld z = std::cos(pi * (i + 0.75L) / (n + 0.5L));
    ld dp = 1;
    for (int it = 0; it < 100; ++it) {
      ld p0 = 1, p1 = 0;
      for (int k = 1; k <= n; ++k) {
        ld p2 = p1;
        p1 = p0;
        p0 = ((2 * k - 1) * z * p1 - (k - 1) * p2) / k;
      }
      dp = n * (z * p0 - p1) / (z * z - 1);
      ld dz = p0 / dp;
      z -= dz;
      if (std::fabs(dz) < 1e-19L) break;
    }
    ld p0 = 1, p1 = 0;
    for (int k = 1; k <= n; ++k) {
      ld p2 = p1;
      p1 = p0;
      p0 = ((2 * k - 1) * z * p1 - (k - 1) * p2) / k;
    }
    dp = n * (z * p0 - p1) / (z * z - 1);
    x[i] = 0.5L * (1 - z);
    w[i] = 1.0L / ((1 - z * z) * dp * dp);  // (2 / ((1-z^2) P'^2)) / 2
  }
}

struct GL {
  std::vector<ld> x32, w32, x24, w24;
  GL() {
    gauss_legendre01(32, x32, w32);
    gauss_legendre01(24, x24, w24);
  }
};
static const GL &gl() {
  static const GL g;
  return g;
}

constexpr int kErfcxPanels = 12;
static ld erfcx_range(ld x) { return -x + std::sqrt(x * x + 46.0L); }

static zl erfcx_integral(zl z) {
  const GL &g = gl();
  const ld S = erfcx_range(z.real());
  zl acc = 0;
  for (int p = 0; p < kErfcxPanels; ++p) {
    const ld lo = S * p / kErfcxPanels, h = S / kErfcxPanels;
    for (size_t i = 0; i < g.x24.size(); ++i) {
      const ld s = lo + h * g.x24[i];
      acc += h * g.w24[i] * std::exp(-s * s - 2.0L * z * s);
    }
  }
  return acc * (2.0L / kSqrtPiL);
}

// the real part alone, with the same operations (im = 0: a real argument)
static ld erfcx_real_part(ld x, ld im) {
  const GL &g = gl();
  const ld S = erfcx_range(x);
  ld acc = 0;
  for (int p = 0; p < kErfcxPanels; ++p) {
    const ld lo = S * p / kErfcxPanels, h = S / kErfcxPanels;
    for (size_t i = 0; i < g.x24.size(); ++i) {
      const ld s = lo + h * g.x24[i];
      const ld e = std::exp(-s * s - 2.0L * x * s);
      acc += h * g.w24[i] * (im == 0 ? e : e * std::cos(2.0L * im * s));
    }
  }
  return acc * (2.0L / kSqrtPiL);
}

static zl erf_integral(zl z) {
  const GL &g = gl();
  zl acc = 0;
  for (size_t i = 0; i < g.x32.size(); ++i) {
    const ld t = g.x32[i];
    acc += g.w32[i] * std::exp(-z * z * (t * t));
  }
  return acc * z * (2.0L / kSqrtPiL);
}

static ld erfcx_real(ld x) {
  return x >= 0 ? erfcx_real_part(x, 0) : 2.0L * std::exp(x * x) - erfcx_real_part(-x, 0);
}

static zl erfc_l(zl z) {
  if (z.real() >= 0.5L) return std::exp(-z * z) * erfcx_integral(z);
  if (z.real() <= -0.5L) return 2.0L - std::exp(-z * z) * erfcx_integral(-z);
  return 1.0L - erf_integral(z);
}

static ld erfi_l(ld y) {
  const GL &g = gl();
  ld acc = 0;
  for (size_t i = 0; i < g.x32.size(); ++i) {
    const ld t = g.x32[i];
    acc += g.w32[i] * std::exp(y * y * t * t);
  }
  return acc * y * (2.0L / kSqrtPiL);
}

// F and H of the images (see build_pgf_table) from these, at y = k0 / 2E.
struct FixedImages {
  ld y, erfi_y;
  explicit FixedImages(ld y) : y(y), erfi_y(erfi_l(y)) {}
  ld tail(ld x) const { return std::exp(y * y - x * x) * erfcx_real_part(x, -y); }   // F(x) for x >= 0.5
  ld H(ld x) const {
    // (F(x) - 1) / x = [-2 sin^2(xy) + sin(2xy) erfi(y) - Re(e^{-2jxy} I(x))] / x,
    // I(x) = (2 / sqrt(pi)) int_0^x exp(-(s - jy)^2) ds  (no cancellation near x = 0)
    if (x > 3.0) return (tail(x) - 1.0L) / x;
    if (x == 0.0) return 2 * y * erfi_y - 2 * std::exp(y * y) / kSqrtPiL;
    const GL &g = gl();
    zl I = 0;
    for (size_t i = 0; i < g.x32.size(); ++i) {
      const ld s = x * g.x32[i];
      const zl d(s, -y);
      I += g.w32[i] * std::exp(-d * d);
    }
    I *= x * 2.0L / kSqrtPiL;
    const ld sxy = std::sin(x * y);
    const ld val = -2 * sxy * sxy + std::sin(2 * x * y) * erfi_y - (std::exp(zl(0, -2 * x * y)) * I).real();
    return val / x;
  }
  ld F(ld x) const { return x >= 0.5 ? tail(x) : 1.0L + x * H(x); }
};

// ---------------------------------------------------------------- quadrature
static double tet14_residual(const double p[6], double r[6]) {
  // exactness on one homogeneous degree-5 barycentric monomial per partition
  static const int parts[6][4] = {{5, 0, 0, 0}, {4, 1, 0, 0}, {3, 2, 0, 0},
                                  {3, 1, 1, 0}, {2, 2, 1, 0}, {2, 1, 1, 1}};
  auto fact = [](int n) {
    double f = 1;
    for (int i = 2; i <= n; ++i) f *= i;
    return f;
  };
  double pts[14][4], w[14];
  int c = 0;
  for (int o = 0; o < 2; ++o) {
    double a = p[2 * o], wa = p[2 * o + 1];
    for (int k = 0; k < 4; ++k, ++c) {
      for (int j = 0; j < 4; ++j) pts[c][j] = j == k ? 1 - 3 * a : a;
      w[c] = wa;
    }
  }
  static const int pr[6][2] = {{0, 1}, {0, 2}, {0, 3}, {1, 2}, {1, 3}, {2, 3}};
  for (int k = 0; k < 6; ++k, ++c) {
    for (int j = 0; j < 4; ++j) pts[c][j] = (j == pr[k][0] || j == pr[k][1]) ? p[4] : 0.5 - p[4];
    w[c] = p[5];
  }
  double nrm = 0;
  for (int e = 0; e < 6; ++e) {
    double exact = 6.0 * fact(parts[e][0]) * fact(parts[e][1]) * fact(parts[e][2]) * fact(parts[e][3]) / fact(8);
    double s = 0;
    for (int i = 0; i < 14; ++i) {
      double m = w[i];
      for (int j = 0; j < 4; ++j) m *= std::pow(pts[i][j], parts[e][j]);
      s += m;
    }
    r[e] = s - exact;
    nrm = std::max(nrm, std::fabs(r[e]));
  }
  return nrm;
}

// Solve the 6x6 moment system of the symmetric 14-point degree-5 rule
// (two (a,a,a,1-3a) orbits and one (b,b,1/2-b,1/2-b) orbit) by Newton's method.
static void solve_tet14(double p[6]) {
  double start[6] = {0.0927, 0.0735, 0.3109, 0.1127, 0.0455, 0.0425};
  std::memcpy(p, start, sizeof(start));
  for (int it = 0; it < 60; ++it) {
    double r[6], J[6][6];
    if (tet14_residual(p, r) < 1e-17) break;
    for (int k = 0; k < 6; ++k) {
      double pp[6], pm[6], rp[6], rm[6];
      std::memcpy(pp, p, sizeof(pp));
      std::memcpy(pm, p, sizeof(pm));
      double h = 1e-7 * std::max(1.0, std::fabs(p[k]));
      pp[k] += h;
      pm[k] -= h;
      tet14_residual(pp, rp);
      tet14_residual(pm, rm);
      for (int e = 0; e < 6; ++e) J[e][k] = (rp[e] - rm[e]) / (2 * h);
    }
    // Gaussian elimination with partial pivoting on J dp = -r
    double A[6][7];
    for (int e = 0; e < 6; ++e) {
      for (int k = 0; k < 6; ++k) A[e][k] = J[e][k];
      A[e][6] = -r[e];
    }
    for (int c = 0; c < 6; ++c) {
      int piv = c;
      for (int e = c + 1; e < 6; ++e)
        if (std::fabs(A[e][c]) > std::fabs(A[piv][c])) piv = e;
      for (int k = 0; k < 7; ++k) std::swap(A[c][k], A[piv][k]);
      for (int e = c + 1; e < 6; ++e) {
        double f = A[e][c] / A[c][c];
        for (int k = c; k < 7; ++k) A[e][k] -= f * A[c][k];
      }
    }
    double dp[6];
    for (int c = 5; c >= 0; --c) {
      double s = A[c][6];
      for (int k = c + 1; k < 6; ++k) s -= A[c][k] * dp[k];
      dp[c] = s / A[c][c];
    }
    for (int k = 0; k < 6; ++k) p[k] += dp[k];
  }
}

void build_quadrature(QuadRules &q) {
  const double al = (5.0 + 3.0 * std::sqrt(5.0)) / 20.0, be = (5.0 - std::sqrt(5.0)) / 20.0;
  for (int i = 0; i < 4; ++i) {
    for (int j = 0; j < 4; ++j) q.tet4[i][j] = i == j ? al : be;
    q.w4[i] = 0.25;
  }
  double p[6];
  solve_tet14(p);
  int c = 0;
  for (int o = 0; o < 2; ++o)
    for (int k = 0; k < 4; ++k, ++c) {
      for (int j = 0; j < 4; ++j) q.tet14[c][j] = j == k ? 1 - 3 * p[2 * o] : p[2 * o];
      q.w14[c] = p[2 * o + 1];
    }
  static const int pr[6][2] = {{0, 1}, {0, 2}, {0, 3}, {1, 2}, {1, 3}, {2, 3}};
  for (int k = 0; k < 6; ++k, ++c) {
    for (int j = 0; j < 4; ++j) q.tet14[c][j] = (j == pr[k][0] || j == pr[k][1]) ? p[4] : 0.5 - p[4];
    q.w14[c] = p[5];
  }
  for (int i = 0; i < 3; ++i) {
    for (int j = 0; j < 3; ++j) q.tri3[i][j] = i == j ? 2.0 / 3.0 : 1.0 / 6.0;
    q.w3[i] = 1.0 / 3.0;
  }
  const double s15 = std::sqrt(15.0);
  const double b1 = (6.0 - s15) / 21.0, b2 = (6.0 + s15) / 21.0;
  const double w1 = (155.0 - s15) / 1200.0, w2 = (155.0 + s15) / 1200.0;
  q.tri7[0][0] = q.tri7[0][1] = q.tri7[0][2] = 1.0 / 3.0;
  q.w7[0] = 9.0 / 40.0;
  c = 1;
  for (int o = 0; o < 2; ++o) {
    double bb = o == 0 ? b1 : b2, ww = o == 0 ? w1 : w2;
    for (int k = 0; k < 3; ++k, ++c) {
      for (int j = 0; j < 3; ++j) q.tri7[c][j] = j == k ? 1 - 2 * bb : bb;
      q.w7[c] = ww;
    }
  }
}

// ---------------------------------------------------------------- Chebyshev fits
// Interpolate f on [lo, hi] at n first-kind Chebyshev nodes; coefficients with
// c[0] halved (so f(t) = sum_k c_k T_k(t)).  A coefficient counts when it
// exceeds thr = max(abs_tol, rel_tol * max|f|); the series has converged when
// the last eight coefficients sit at that noise level.  The kept degree is
// the last counting coefficient.  Returns the degree, or -1 if neither 48 nor
// 96 nodes converge within maxdeg.
// cos(pi k (j + 1/2) / n), j < n, at k n + j for n = 48 and 96: the nodes
// (k = 1) and the transform
struct CosTable {
  std::vector<ld> c48, c96;
  CosTable() {
    const ld pi = 3.141592653589793238462643383279502884L;
    for (int n : {48, 96})
      for (int k = 0; k < n; ++k)
        for (int j = 0; j < n; ++j) (n == 48 ? c48 : c96).push_back(std::cos(pi * k * (j + 0.5L) / n));
  }
};
static const CosTable &cosines() {
  static const CosTable c;
  return c;
}

template <class F>
static int cheb_fit(F f, double lo, double hi, double abs_tol, double rel_tol, double *out, int maxdeg) {
  for (int n : {48, 96}) {
    const std::vector<ld> &cs = n == 48 ? cosines().c48 : cosines().c96;
    ld fx[96];
    double c[96];
    double fmax = 0;
    for (int j = 0; j < n; ++j) {
      const double t = (double)cs[n + j];
      fx[j] = f(lo + 0.5 * (t + 1) * (hi - lo));
      fmax = std::max(fmax, (double)std::fabs(fx[j]));
    }
    for (int k = 0; k < n; ++k) {
      ld s = 0;
      for (int j = 0; j < n; ++j) s += fx[j] * cs[(size_t)k * n + j];
      c[k] = (double)(2.0L * s / n);
    }
    c[0] *= 0.5;
    const double thr = std::max(abs_tol, rel_tol * fmax);
    double tailmax = 0;
    for (int k = n - 8; k < n; ++k) tailmax = std::max(tailmax, std::fabs(c[k]));
    int deg = 0;
    for (int k = n - 1; k >= 1; --k)
      if (std::fabs(c[k]) > thr) {
        deg = k;
        break;
      }
    if (tailmax <= 16 * thr && deg <= maxdeg) {
      for (int k = 0; k <= deg; ++k) out[k] = c[k];
      for (int k = deg + 1; k <= maxdeg; ++k) out[k] = 0;
      return deg;
    }
  }
  return -1;
}

// Run body(i) for i in [0, n) on up to 16 host threads.
template <class Fn>
static void parallel_for(int n, Fn body) {
  const int nth = std::max(1, std::min<int>({16, n, (int)std::thread::hardware_concurrency()}));
  std::atomic<int> next(0);
  (void)cosines();   // (made here, not by the first thread to need them)
  auto work = [&]() {
    for (int i = next++; i < n; i = next++) body(i);
  };
  std::vector<std::thread> th;
  th.reserve(nth);
  try {
    for (int k = 1; k < nth; ++k) th.emplace_back(work);
  } catch (const std::system_error &) {   // no more threads to be had: fewer do it
  }
  work();
  for (auto &t : th) t.join();
}

// ---------------------------------------------------------------- Ewald tables
std::string build_pgf_table(PgfTable &tab, double a, double b, double zspan, double lambda, double theta,
                            double phi, double *wood_margin, PgfTerms terms) {
  std::memset(&tab, 0, sizeof(tab));
  const double k0 = 2 * kPi / lambda;
  const double kx = k0 * std::sin(theta) * std::cos(phi), ky = k0 * std::sin(theta) * std::sin(phi);
  const double E = std::sqrt(kPi / (a * b));
  const double y = k0 / (2 * E);
  tab.a = a;
  tab.b = b;
  tab.inv_a = 1 / a;
  tab.inv_b = 1 / b;
  tab.E = E;
  tab.k0 = k0;
  tab.kx = kx;
  tab.ky = ky;
  tab.two_pi_a = 2 * kPi / a;
  tab.two_pi_b = 2 * kPi / b;
  for (int m0 = -1; m0 <= 1; ++m0)
    for (int n0 = -1; n0 <= 1; ++n0) {
      double ph = -(kx * m0 * a + ky * n0 * b);
      tab.ph0re[(m0 + 1) * 3 + (n0 + 1)] = std::cos(ph);
      tab.ph0im[(m0 + 1) * 3 + (n0 + 1)] = std::sin(ph);
    }

  // Wood-anomaly margin over the non-specular orders
  double margin = 1e300;
  for (int p = -kPgfM; p <= kPgfM; ++p)
    for (int q = -kPgfM; q <= kPgfM; ++q) {
      if (p == 0 && q == 0) continue;
      double tx = kx + 2 * kPi * p / a, ty = ky + 2 * kPi * q / b;
      margin = std::min(margin, std::sqrt(std::fabs(tx * tx + ty * ty - k0 * k0)) / k0);
    }
  margin = std::min(margin, std::cos(theta));
  *wood_margin = margin;
  if (margin < 0.02) return "";  // the caller reports the anomaly; no tables near gamma = 0

  // Accuracy of the tables: a term is dropped when it stays below 1e-16 of
  // g_p's size at the largest in-cell separation, and the fits resolve every
  // term to 1e-15 (absolute) / 1e-14 (relative).  The lattice sum then stays
  // within a few 1e-13 of its converged value (relative), three orders of
  // magnitude inside what the fill is held to (1e-10 of each Z entry).
  const double G = 1.0 / (4 * kPi * std::sqrt(a * a + b * b + zspan * zspan));
  const double sig = 1e-16 * G;
  const double fit_abs = 1e-15, fit_rel = 1e-14;

  // F(x) = (2x / sqrt(pi)) int_1^inf exp(-x^2 s^2 + y^2 / s^2) ds, and H = (F - 1) / x with
  // the n = 0 term erfc(x) - 1 = -erf(x) taken out: no cancellation near x = 0
  const ld yl = y;
  const bool fixed = terms == PgfTerms::fixed;
  const FixedImages fim(yl);
  auto Fx = [&](double x) -> ld {
    return fixed ? fim.F(x) : std::erfc((ld)x) + 2 * (ld)x / kSqrtPiL * tail_sum(x, yl * yl, 0, 1);
  };
  auto Hx = [&](double x) -> ld {
    if (fixed) return fim.H(x);
    const ld xl = x, e0 = x == 0.0 ? 2 / kSqrtPiL : std::erf(xl) / xl;
    return 2 / kSqrtPiL * tail_sum(xl, yl * yl, 0, 1) - e0;
  };

  // ---- spatial images: significance cut first
  struct ImgJob {
    int m, n;
    double xlo, xhi;
    bool touching;
  };
  std::vector<ImgJob> jobs;
  for (int m = -kPgfM; m <= kPgfM; ++m)
    for (int n = -kPgfM; n <= kPgfM; ++n) {
      double dxlo = std::max(0.0, (std::abs(m) - 0.5) * a), dylo = std::max(0.0, (std::abs(n) - 0.5) * b);
      double dxhi = (std::abs(m) + 0.5) * a, dyhi = (std::abs(n) + 0.5) * b;
      double Rlo = std::sqrt(dxlo * dxlo + dylo * dylo) * (1 - 1e-9);
      double Rhi = std::sqrt(dxhi * dxhi + dyhi * dyhi + zspan * zspan) * (1 + 1e-9);
      double xlo = Rlo * E, xhi = Rhi * E;
      bool touching_class = std::abs(m) <= 1 && std::abs(n) <= 1;
      if (!touching_class && Rlo > 0 && std::exp(y * y - xlo * xlo) / (4 * kPi * Rlo) < sig) continue;
      jobs.push_back({m, n, xlo, xhi, touching_class});
    }
  tab.nimg = (int)jobs.size();
  // ---- spectral modes, K_pq as a function of w = (z E)^2 on [0, (zspan E)^2]
  const double wmax = std::max(1e-30, zspan * E * zspan * E) * (1 + 1e-9);
  tab.ws = 2.0 / wmax;
  const auto kt2_of = [&](int idx) {
    const int p = idx / kPgfSide - kPgfM, q = idx % kPgfSide - kPgfM;
    const double tx = kx + 2 * kPi * p / a, ty = ky + 2 * kPi * q / b;
    return tx * tx + ty * ty;
  };

  // The fits, each distinct one once: an image's depends on |m|, |n| alone, an
  // order's on |k_t|^2.
  const auto same_image = [&](int i, int k) {
    return std::abs(jobs[k].m) == std::abs(jobs[i].m) && std::abs(jobs[k].n) == std::abs(jobs[i].n);
  };
  int first_img[kPgfTerms], first_mode[kPgfTerms];
  enum Fit { FIT_F, FIT_H, FIT_K };
  std::vector<std::pair<Fit, int>> todo;
  for (int i = 0; i < kPgfTerms; ++i) {   // (the propagating orders, which take longest, first)
    first_mode[i] = 0;
    while (kt2_of(first_mode[i]) != kt2_of(i)) ++first_mode[i];
    if (first_mode[i] == i && kt2_of(i) <= k0 * k0) todo.push_back({FIT_K, i});
  }
  for (int i = 0; i < tab.nimg; ++i) {
    int k = 0;
    while (!same_image(i, k)) ++k;
    first_img[i] = k;
    if (k < i) continue;
    todo.push_back({FIT_F, i});
    tab.img[i].hdeg = -1;
    if (jobs[i].touching) todo.push_back({FIT_H, i});
  }
  for (int i = 0; i < kPgfTerms; ++i)
    if (first_mode[i] == i && kt2_of(i) > k0 * k0) todo.push_back({FIT_K, i});
  std::atomic<bool> bad_image(false), bad_mode(false);
  const auto fit_image = [&](Fit fit, int i) {
    const ImgJob &jb = jobs[i];
    PgfImage &im = tab.img[i];
    int &deg = fit == FIT_H ? im.hdeg : im.deg;
    if (fit == FIT_H) deg = cheb_fit(Hx, jb.xlo, jb.xhi, 0.0, fit_rel, im.h, kPgfMaxDeg - 1);
    else deg = cheb_fit(Fx, jb.xlo, jb.xhi, fit_abs, fit_rel, im.f, kPgfMaxDeg - 1);
    if (deg < 0) bad_image = true;
  };
  const auto fit_mode = [&](int idx) {
    const double kt2 = kt2_of(idx);
    PgfMode &md = tab.mode[idx];
    md.deg = -1;
    if (kt2 > k0 * k0) {
      double gam = std::sqrt(kt2 - k0 * k0);
      double u = gam / (2 * E);
      double pref = 1.0 / (4 * a * b * gam);
      auto K = [&](double w) -> ld {
        const ld v = std::sqrt(std::max(0.0L, (ld)w)), ul = u;
        if (fixed) {
          const ld e = std::exp(-ul * ul - v * v);
          return (ld)pref * (e * erfcx_real(ul + v) + e * erfcx_real(ul - v));
        }
        return (ld)pref * (std::exp(2 * ul * v) * std::erfc(ul + v) + std::exp(-2 * ul * v) * std::erfc(ul - v));
      };
      if ((double)K(0.0) < sig) return;  // K falls with z; deg stays -1
      md.deg = cheb_fit(K, 0.0, wmax, sig, fit_rel, md.kre, kPgfMaxDeg - 1);
      if (md.deg < 0) bad_mode = true;
    } else {
      // propagating order, gamma = +j beta: the whole transform e^{-j beta z} / (2 j beta)
      // less its part beyond the split, int_E^inf exp(-z^2 s^2 + beta^2 / 4 s^2) / (2 sqrt(pi) s^2) ds
      const double beta = std::sqrt(k0 * k0 - kt2);
      const ld bb = beta / (2 * E), area = a * b;
      const zl pref = 1.0L / (4.0L * a * b * zl(0, beta));
      // the same by erfc of complex arguments, whose values serve both parts' fits
      std::pair<double, zl> seen[48 + 96];
      int nseen = 0;
      const auto Kc = [&](double w) -> zl {
        for (int i = 0; i < nseen; ++i)
          if (seen[i].first == w) return seen[i].second;
        const ld v = std::sqrt(std::max(0.0L, (ld)w));
        const zl e1 = std::exp(zl(0, 2 * bb * v)), e2 = std::exp(zl(0, -2 * bb * v));
        const zl K = pref * (e1 * erfc_l(zl(v, bb)) + e2 * erfc_l(zl(-v, bb)));
        if (nseen < 48 + 96) seen[nseen++] = {w, K};
        return K;
      };
      md.cplx = 1;
      const int d1 = cheb_fit(
          [&](double w) -> ld {
            if (fixed) return Kc(w).real();
            const ld v = std::sqrt(std::max(0.0L, (ld)w));
            return -(std::sin(2 * bb * v) / (2 * beta) + tail_sum(v, bb * bb, 1, 0) / (2 * kSqrtPiL * E)) / area;
          },
          0.0, wmax, sig, fit_rel, md.kre, kPgfMaxDeg - 1);
      const int d2 = cheb_fit(
          [&](double w) -> ld {
            if (fixed) return Kc(w).imag();
            return -std::cos(2 * bb * std::sqrt(std::max(0.0L, (ld)w))) / (2 * beta * area);
          },
          0.0, wmax, sig, fit_rel, md.kim, kPgfMaxDeg - 1);
      if (d1 < 0 || d2 < 0) bad_mode = true;
      md.deg = std::max(d1, d2);
    }
  };
  const auto fit = [&](int i) {
    if (todo[i].first == FIT_K) fit_mode(todo[i].second);
    else fit_image(todo[i].first, todo[i].second);
  };
  // (the quadratures take 100 ms of one thread, the series 2)
  if (fixed) parallel_for((int)todo.size(), fit);
  else for (int i = 0; i < (int)todo.size(); ++i) fit(i);
  if (bad_image) return "lattice-sum table: spatial fit did not converge";
  if (bad_mode) return "lattice-sum table: spectral fit did not converge";
  for (int i = 0; i < tab.nimg; ++i) {
    PgfImage &im = tab.img[i];
    if (first_img[i] != i) im = tab.img[first_img[i]];
    im.xa = jobs[i].xlo;
    im.xs = 2.0 / (jobs[i].xhi - jobs[i].xlo);
    im.m = jobs[i].m;
    im.n = jobs[i].n;
    double ph = kx * im.m * a + ky * im.n * b;
    im.cre = std::cos(ph) / (4 * kPi);
    im.cim = std::sin(ph) / (4 * kPi);
  }
  for (int i = 0; i < kPgfTerms; ++i) {
    if (first_mode[i] != i) tab.mode[i] = tab.mode[first_mode[i]];
    tab.mode[i].p = i / kPgfSide - kPgfM;
    tab.mode[i].q = i % kPgfSide - kPgfM;
  }
  return "";
}

// ---------------------------------------------------------------- packing
// An integer field of the packed table: its value in the low 32 bits of the
// double slot (the device reads the register half, no conversion).
static double ibits(int v, int hi = 0) {
  const uint64_t u = (uint64_t)(uint32_t)hi << 32 | (uint32_t)v;
  double d;
  std::memcpy(&d, &u, sizeof d);
  return d;
}

// Coefficients of a Chebyshev series, the highest degree first and the degree
// rounded up to an even K: as they are, or of its monomials.
static std::vector<double> series_coeffs(const std::vector<ld> &c, bool mono) {
  const int n = (int)c.size(), K = n & ~1;   // degree n - 1, rounded up to even
  std::vector<ld> m(c);
  if (mono) {
    std::vector<ld> T0(n, 0), T1(n, 0), T2(n, 0);   // T_{k-1}, T_k, T_{k+1}
    m.assign(n, 0);
    T1[0] = 1;
    for (int k = 0; k < n; ++k) {
      for (int i = 0; i <= k; ++i) m[i] += c[k] * T1[i];
      for (int i = 0; i < n; ++i) T2[i] = (i ? (k ? 2 : 1) * T1[i - 1] : 0) - (k ? T0[i] : 0);
      T0 = T1;
      T1 = T2;
    }
  }
  std::vector<double> out(K + 1, 0.0);
  for (int k = 0; k < n; ++k) out[K - k] = (double)m[k];
  return out;
}

static std::vector<ld> cheb_of(const double *c, int deg) { return std::vector<ld>(c, c + std::max(0, deg) + 1); }

// What the rounding of a series' monomials may reach (sum |a_k|) and the same
// of its Chebyshev coefficients.
static double abs_sum(const std::vector<ld> &c, bool mono) {
  double s = 0;
  for (double v : series_coeffs(c, mono)) s += std::fabs(v);
  return s;
}

void pack_pgf_table(const PgfTable &tab, std::vector<double> &out) {
  const PgfImage *img[kPgfM + 1][2 * kPgfM + 1] = {};   // [m][n + kPgfM], m >= 0
  int rown[kPgfM + 1] = {};
  for (int i = 0; i < tab.nimg; ++i)
    if (tab.img[i].m >= 0) img[tab.img[i].m][tab.img[i].n + kPgfM] = &tab.img[i];
  for (int m = 0; m <= kPgfM; ++m)
    while (rown[m] <= kPgfM && img[m][kPgfM + rown[m]]) ++rown[m];
  const auto mode = [&](int p, int q) { return &tab.mode[(p + kPgfM) * kPgfSide + q + kPgfM]; };
  const auto kre = [&](int p, int q) {
    const PgfMode *md = mode(p, q);
    return md->deg < 0 ? std::vector<ld>{0} : cheb_of(md->kre, md->deg);
  };
  // sums and differences of the series of (p, q) and (p, -q)
  const auto pair = [&](int p, int q, int sign) {
    std::vector<ld> u = kre(p, q), v = kre(p, -q);
    u.resize(std::max(u.size(), v.size()), 0);
    for (size_t k = 0; k < v.size(); ++k) u[k] += sign * v[k];
    return u;
  };

  // Monomials cost one FMA per degree against an addition more, and round by
  // up to sum |a_k| eps where the Chebyshev form does by sum |c_k| eps.  They
  // are taken where that stays a few eps of g_p: every series near R = 0 and
  // every order within 8 of its Chebyshev sum, the images further off
  // (|F| / 4 pi R, all of them) within 32 of g_p at the largest in-cell
  // separation.  Measured over cells of 20-600 nm at 300-1500 nm: orders
  // 1-3, images 4-20 times, while the structure's height is below 2.3 periods;
  // taller cells and periods above the wavelength keep the Chebyshev form.
  const double zspan = std::sqrt(2.0 / tab.ws) / tab.E;
  const double G = 1.0 / (4 * kPi * std::sqrt(tab.a * tab.a + tab.b * tab.b + zspan * zspan));
  bool mono = true;
  double far = 0;
  for (int m = 0; m <= kPgfM; ++m)
    for (int n = 0; n < rown[m]; ++n) {
      const PgfImage &im = *img[m][kPgfM + n];
      const std::vector<ld> f = cheb_of(im.f, im.deg);
      if (im.xa > 0) far += (m ? 2 : 1) * (n ? 2 : 1) * abs_sum(f, true) * tab.E / (4 * kPi * im.xa);
      else mono = mono && abs_sum(f, true) <= 8 * abs_sum(f, false);
      if (im.hdeg >= 0) {
        const std::vector<ld> h = cheb_of(im.h, im.hdeg);
        mono = mono && abs_sum(h, true) <= 8 * abs_sum(h, false);
      }
    }
  mono = mono && far <= 32 * G;
  for (int idx = 0; idx < kPgfTerms && mono; ++idx) {
    const PgfMode &md = tab.mode[idx];
    if (md.deg < 0) continue;
    mono = abs_sum(cheb_of(md.kre, md.deg), true) <= 8 * abs_sum(cheb_of(md.kre, md.deg), false);
    if (md.cplx) mono = mono && abs_sum(cheb_of(md.kim, md.deg), true) <= 8 * abs_sum(cheb_of(md.kim, md.deg), false);
  }

  out.assign(kPackImages, 0.0);
  const double hdr[10] = {tab.E, tab.a, tab.b, tab.inv_a, tab.inv_b, tab.kx / kPi, tab.ky / kPi, ibits(mono ? 0 : 1), 0.0,
                          tab.ws * tab.E * tab.E};
  for (int i = 0; i < 10; ++i) out[i] = hdr[i];
  for (int i = 0; i < 9; ++i) {
    out[10 + i] = tab.ph0re[i];
    out[19 + i] = tab.ph0im[i];
  }
  const auto series = [&](const std::vector<ld> &c, int hi = 0) {
    const std::vector<double> e = series_coeffs(c, mono);
    out.push_back(ibits((int)e.size() - 1, hi));
    out.insert(out.end(), e.begin(), e.end());
  };
  for (int m = 0; m <= kPgfM; ++m) {
    out[kPackRows + m] = ibits(rown[m]);
    for (int n = 0; n < rown[m]; ++n) {
      const PgfImage &im = *img[m][kPgfM + n], &in = *img[m][kPgfM - n];
      const size_t start = out.size();
      // the fit's argument t = (x - xa) xs - 1 with x = E R, stored as t = R (E xs) - (xa xs + 1)
      out.insert(out.end(), {tab.E * im.xs, -(im.xa * im.xs + 1.0), im.cre, im.cim, in.cre, in.cim});
      series(cheb_of(im.f, im.deg));
      const int K = (int)(out.size() - start) - 8;
      if (im.hdeg >= 0) series(cheb_of(im.h, im.hdeg));
      out[start + 6] = ibits(K, (int)(out.size() - start));
    }
  }
  // rows p of the orders, the last first: [q_max | differences], K_p0, then S_q (and D_q)
  int plo = 0, phi = 0;
  for (int idx = 0; idx < kPgfTerms; ++idx)
    if (tab.mode[idx].deg >= 0) {
      plo = std::min(plo, idx / kPgfSide - kPgfM);
      phi = std::max(phi, idx / kPgfSide - kPgfM);
    }
  out[8] = ibits((int)out.size(), (plo + 8) | (phi + 8) << 8);
  for (int p = phi; p >= plo; --p) {
    int nq = 0;
    bool odd = false;
    for (int q = 1; q <= kPgfM; ++q) {
      if (mode(p, q)->deg >= 0 || mode(p, -q)->deg >= 0) nq = q;
      for (ld v : pair(p, q, -1)) odd = odd || v != 0;
    }
    out.push_back(ibits(nq, odd ? 1 : 0));
    out.push_back(0.0);
    series(kre(p, 0));
    for (int q = 1; q <= nq; ++q) {
      if (!odd) {
        series(pair(p, q, 1));
        continue;
      }
      // the sum's and the difference's coefficients interleaved
      const std::vector<double> e = series_coeffs(pair(p, q, 1), mono), d = series_coeffs(pair(p, q, -1), mono);
      out.insert(out.end(), {ibits((int)e.size() - 1), 0.0});
      for (size_t k = 0; k < e.size(); ++k) out.insert(out.end(), {e[k], d[k]});
    }
  }
  // the imaginary parts of the propagating orders
  int nprop = 0;
  const size_t props = out.size();
  for (int idx = 0; idx < kPgfTerms; ++idx) {
    const PgfMode &md = tab.mode[idx];
    if (md.deg < 0 || !md.cplx) continue;
    ++nprop;
    out.push_back(ibits(md.p, md.q));
    out.push_back(0.0);
    series(cheb_of(md.kim, md.deg));
  }
  out[28] = ibits((int)props, nprop);
  out.insert(out.end(), 4, 0.0);   // a series reads one pair past its end
}

size_t pgf_listed_doubles(const PgfTable &tab) {
  const auto pad4 = [](int n) { return (size_t)((n + 3) & ~3); };
  const auto listed = [&](int deg) { return 4 + pad4((int)pad4(deg) + 1); };
  size_t n = 128;
  for (int i = 0; i < tab.nimg; ++i) n += 4 + listed(tab.img[i].deg) + (tab.img[i].hdeg >= 0 ? listed(tab.img[i].hdeg) : 0);
  for (const PgfMode &md : tab.mode)
    if (md.deg >= 0) n += listed(md.deg) + (md.cplx ? listed(md.deg) - 4 : 0);
  return n;
}

void pack_pgf_fixed(const PgfTable &tab, std::vector<double> &out) {
  out.assign(kFixedRecords, 0.0);
  const double hdr[10] = {tab.E, tab.a, tab.b, tab.inv_a, tab.inv_b, tab.kx, tab.ky, tab.two_pi_a, tab.two_pi_b, tab.ws};
  for (int i = 0; i < 10; ++i) out[i] = hdr[i];
  for (int i = 0; i < 9; ++i) {
    out[10 + i] = tab.ph0re[i];
    out[19 + i] = tab.ph0im[i];
  }
  // a series without its leading zeros, which add nothing to the recurrence, but
  // of an even degree of 4 at the least, and with the third coefficient less the
  // first, as the recurrence takes it; the record's length beside the degree
  const auto series = [&](const double *c, int deg, size_t start) {
    while (deg > 4 && c[deg] == 0.0) --deg;
    deg = std::max(4, (deg + 1) & ~1);
    const auto at = [&](int k) { return k <= kPgfMaxDeg ? c[k] : 0.0; };
    const size_t head = out.size();
    out.insert(out.end(), {0.0, at(deg), at(deg - 1), at(deg - 2) - at(deg)});
    for (int k = deg - 3; k >= 0; --k) out.push_back(c[k]);
    while (out.size() & 3) out.push_back(0.0);
    out[head] = ibits(deg, (int)(out.size() - start));
  };
  int mmax = 0, nmax[kPgfM + 1] = {};
  for (int i = 0; i < tab.nimg; ++i) {   // (in the order of (m, n))
    const PgfImage &im = tab.img[i];
    mmax = std::max(mmax, im.m);
    if (im.m >= 0) nmax[im.m] = std::max(nmax[im.m], im.n);
    // the fit's argument t = (x - xa) xs - 1 with x = E R, stored as t = R (E xs) - (xa xs + 1)
    const size_t start = out.size();
    out.insert(out.end(), {tab.E * im.xs, -(im.xa * im.xs + 1.0), im.cre, im.cim});
    series(im.f, im.deg, start);
  }
  out[28] = ibits(mmax);
  for (int m = 0; m <= kPgfM; ++m) out[kFixedNmax + m] = ibits(nmax[m]);
  for (int p = 0; p < kPgfSide; ++p) {
    int any = 0, cplx = 0;
    for (int q = 0; q < kPgfSide; ++q) {
      const PgfMode &md = tab.mode[p * kPgfSide + q];
      if (md.deg < 0) continue;
      any |= 1 << q;
      if (md.cplx) cplx |= 1 << q;
      series(md.kre, md.deg, out.size());
      if (md.cplx) series(md.kim, md.deg, out.size());
    }
    out[kFixedRows + p] = ibits(any, cplx);
  }
  out.insert(out.end(), 16, 0.0);   // (read ahead past the last record)
}

}  // namespace vie
