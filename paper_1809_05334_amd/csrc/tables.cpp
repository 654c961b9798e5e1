// Host tables of libvie: quadrature rules, special functions and the per-fill
// Ewald lattice-sum tables (Sec. 2.2, Eqs. 3-4 and the Ewald split).
#include <algorithm>
#include <cmath>
#include <cstring>
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
// (16-18 ms on 16 threads), the tables now take 2 ms on one.
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
// cos(pi i / 2n), i < 4n, for n = 48 and 96: the nodes and the transform
struct CosTable {
  std::vector<ld> c48, c96;
  CosTable() {
    const ld pi = 3.141592653589793238462643383279502884L;
    for (int i = 0; i < 4 * 48; ++i) c48.push_back(std::cos(pi * i / (2 * 48)));
    for (int i = 0; i < 4 * 96; ++i) c96.push_back(std::cos(pi * i / (2 * 96)));
  }
};

template <class F>
static int cheb_fit(F f, double lo, double hi, double abs_tol, double rel_tol, double *out, int maxdeg) {
  static const CosTable cosines;
  for (int n : {48, 96}) {
    const std::vector<ld> &cs = n == 48 ? cosines.c48 : cosines.c96;
    ld fx[96];
    double c[96];
    double fmax = 0;
    for (int j = 0; j < n; ++j) {
      const double t = (double)cs[2 * j + 1];
      fx[j] = f(lo + 0.5 * (t + 1) * (hi - lo));
      fmax = std::max(fmax, (double)std::fabs(fx[j]));
    }
    for (int k = 0; k < n; ++k) {
      ld s = 0;
      for (int j = 0, i = k; j < n; ++j) {
        s += fx[j] * cs[i];   // i = k (2j + 1) mod 4n
        i += 2 * k;
        if (i >= 4 * n) i -= 4 * n;
      }
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

// ---------------------------------------------------------------- Ewald tables
std::string build_pgf_table(PgfTable &tab, double a, double b, double zspan, double lambda, double theta,
                            double phi, double *wood_margin) {
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
  auto Fx = [&](double x) -> ld { return std::erfc((ld)x) + 2 * (ld)x / kSqrtPiL * tail_sum(x, yl * yl, 0, 1); };
  auto Hx = [&](double x) -> ld {
    const ld xl = x, e0 = x == 0.0 ? 2 / kSqrtPiL : std::erf(xl) / xl;
    return 2 / kSqrtPiL * tail_sum(xl, yl * yl, 0, 1) - e0;
  };

  // ---- spatial images: significance cut first, then the fits in parallel
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
  bool bad = false;
  for (int i = 0; i < tab.nimg; ++i) {
    const ImgJob &jb = jobs[i];
    PgfImage &im = tab.img[i];
    // the fit depends on |m|, |n| alone: an earlier image with the same gives it
    for (int k = 0; k < i; ++k)
      if (std::abs(jobs[k].m) == std::abs(jb.m) && std::abs(jobs[k].n) == std::abs(jb.n)) {
        im = tab.img[k];
        break;
      }
    if (im.xs == 0) {
      im.xa = jb.xlo;
      im.xs = 2.0 / (jb.xhi - jb.xlo);
      im.deg = cheb_fit(Fx, jb.xlo, jb.xhi, fit_abs, fit_rel, im.f, kPgfMaxDeg - 1);
      im.hdeg = -1;
      if (jb.touching) im.hdeg = cheb_fit(Hx, jb.xlo, jb.xhi, 0.0, fit_rel, im.h, kPgfMaxDeg - 1);
      if (im.deg < 0 || (jb.touching && im.hdeg < 0)) bad = true;
    }
    im.m = jb.m;
    im.n = jb.n;
    double ph = kx * jb.m * a + ky * jb.n * b;
    im.cre = std::cos(ph) / (4 * kPi);
    im.cim = std::sin(ph) / (4 * kPi);
  }
  if (bad) return "lattice-sum table: spatial fit did not converge";

  // ---- spectral modes, K_pq as a function of w = (z E)^2 on [0, (zspan E)^2]
  const double wmax = std::max(1e-30, zspan * E * zspan * E) * (1 + 1e-9);
  tab.ws = 2.0 / wmax;
  for (int idx = 0; idx < kPgfTerms; ++idx) {
      const int p = idx / kPgfSide - kPgfM, q = idx % kPgfSide - kPgfM;
      double tx = kx + 2 * kPi * p / a, ty = ky + 2 * kPi * q / b;
      double kt2 = tx * tx + ty * ty;
      PgfMode &md = tab.mode[(p + kPgfM) * kPgfSide + (q + kPgfM)];
      md.deg = -1;
      md.p = p;
      md.q = q;
      if (kt2 > k0 * k0) {
        double gam = std::sqrt(kt2 - k0 * k0);
        double u = gam / (2 * E);
        double pref = 1.0 / (4 * a * b * gam);
        auto K = [&](double w) -> ld {
          const ld v = std::sqrt(std::max(0.0L, (ld)w)), ul = u;
          return (ld)pref * (std::exp(2 * ul * v) * std::erfc(ul + v) + std::exp(-2 * ul * v) * std::erfc(ul - v));
        };
        if ((double)K(0.0) < sig) continue;  // K falls with z; deg stays -1
        md.cplx = 0;
        md.deg = cheb_fit(K, 0.0, wmax, sig, fit_rel, md.kre, kPgfMaxDeg - 1);
        if (md.deg < 0) bad = true;
      } else {
        // propagating order, gamma = +j beta: the whole transform e^{-j beta z} / (2 j beta)
        // less its part beyond the split, int_E^inf exp(-z^2 s^2 + beta^2 / 4 s^2) / (2 sqrt(pi) s^2) ds
        const double beta = std::sqrt(k0 * k0 - kt2);
        const ld bb = beta / (2 * E), area = a * b;
        md.cplx = 1;
        const int d1 = cheb_fit(
            [&](double w) {
              const ld v = std::sqrt(std::max(0.0L, (ld)w));
              return -(std::sin(2 * bb * v) / (2 * beta) + tail_sum(v, bb * bb, 1, 0) / (2 * kSqrtPiL * E)) / area;
            },
            0.0, wmax, sig, fit_rel, md.kre, kPgfMaxDeg - 1);
        const int d2 = cheb_fit(
            [&](double w) { return -std::cos(2 * bb * std::sqrt(std::max(0.0L, (ld)w))) / (2 * beta * area); }, 0.0,
            wmax, sig, fit_rel, md.kim, kPgfMaxDeg - 1);
        if (d1 < 0 || d2 < 0) bad = true;
        md.deg = std::max(d1, d2);
      }
  }
  if (bad) return "lattice-sum table: spectral fit did not converge";
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

void pack_pgf_table(const PgfTable &tab, std::vector<double> &out) {
  auto pad4 = [](int n) { return (n + 3) & ~3; };
  out.assign(kPackImages, 0.0);
  const double hdr[10] = {tab.E, tab.a, tab.b, tab.inv_a, tab.inv_b, tab.kx, tab.ky, tab.two_pi_a, tab.two_pi_b, tab.ws};
  for (int i = 0; i < 10; ++i) out[i] = hdr[i];
  for (int i = 0; i < 9; ++i) {
    out[10 + i] = tab.ph0re[i];
    out[19 + i] = tab.ph0im[i];
  }
  out[28] = ibits(tab.nimg);
  for (int i = 0; i < tab.nimg; ++i) {
    const PgfImage &im = tab.img[i];
    const int K = pad4(im.deg), HK = im.hdeg >= 0 ? pad4(im.hdeg) : -1;
    const size_t start = out.size();
    // the fit's argument t = (x - xa) xs - 1 with x = E R, stored as t = R (E xs) - (xa xs + 1)
    out.insert(out.end(), {tab.E * im.xs, -(im.xa * im.xs + 1.0), im.cre, im.cim, ibits(im.m), ibits(im.n), ibits(K), 0.0});
    for (int k = 0; k < pad4(K + 1); ++k) out.push_back(k <= im.deg ? im.f[k] : 0.0);
    if (HK >= 0) {
      out.insert(out.end(), {ibits(HK), 0.0, 0.0, 0.0});
      for (int k = 0; k < pad4(HK + 1); ++k) out.push_back(k <= im.hdeg ? im.h[k] : 0.0);
    }
    out[start + 7] = ibits((int)(out.size() - start));
  }
  for (int idx = 0; idx < kPgfTerms; ++idx) {
    const PgfMode &md = tab.mode[idx];
    if (md.deg < 0) continue;
    const int K = pad4(md.deg);
    out[32 + idx] = ibits((int)out.size(), K | (md.cplx ? 1 << 16 : 0));
    out.insert(out.end(), {ibits(K), ibits(md.cplx), 0.0, 0.0});
    for (int k = 0; k < pad4(K + 1); ++k) out.push_back(k <= md.deg ? md.kre[k] : 0.0);
    if (md.cplx)
      for (int k = 0; k < pad4(K + 1); ++k) out.push_back(k <= md.deg ? md.kim[k] : 0.0);
  }
  // each row's range of q with a mode, so that a pass over the grid skips the rest
  for (int p = 0; p < kPgfSide; ++p) {
    int lo = kPgfSide, hi = -1;
    for (int q = 0; q < kPgfSide; ++q)
      if (tab.mode[p * kPgfSide + q].deg >= 0) {
        lo = std::min(lo, q);
        hi = std::max(hi, q);
      }
    out[kPackRows + p] = ibits(hi < 0 ? 0 : lo | (hi + 1) << 8);
  }
}

}  // namespace vie
