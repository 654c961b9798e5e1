// Device helpers of libvie: complex arithmetic, Chebyshev evaluation, the
// Ewald periodic Green's function (Sec. 2.2, Eqs. 3-4) from the per-fill
// tables, and the closed-form 1/R and R potentials of a triangle and a
// tetrahedron (extracted singular part of the kernel).
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "common.h"

namespace vie {

struct dz {
  double re, im;
};
// complex FP32: storage of the mixed-precision Z and of FP32 block factors
struct fz {
  float re, im;
};
__device__ __forceinline__ dz mk(double r, double i) { return dz{r, i}; }
__device__ __forceinline__ dz operator+(dz a, dz b) { return dz{a.re + b.re, a.im + b.im}; }
__device__ __forceinline__ dz operator-(dz a, dz b) { return dz{a.re - b.re, a.im - b.im}; }
__device__ __forceinline__ dz operator*(dz a, dz b) {
  return dz{fma(a.re, b.re, -a.im * b.im), fma(a.re, b.im, a.im * b.re)};
}
__device__ __forceinline__ dz operator*(double s, dz a) { return dz{s * a.re, s * a.im}; }
__device__ __forceinline__ dz operator*(dz a, double s) { return dz{s * a.re, s * a.im}; }
__device__ __forceinline__ dz conjz(dz a) { return dz{a.re, -a.im}; }
// acc += a * s (s real)
__device__ __forceinline__ void axpy(dz &acc, double s, dz a) {
  acc.re = fma(s, a.re, acc.re);
  acc.im = fma(s, a.im, acc.im);
}
// 64-bit DPP lane move (CTRL: a row-local permutation) and lane read, as two
// 32-bit halves
template <int CTRL>
__device__ __forceinline__ unsigned long long dpp64(unsigned long long v) {
  const int lo = __builtin_amdgcn_update_dpp((int)(unsigned)v, (int)(unsigned)v, CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp((int)(unsigned)(v >> 32), (int)(unsigned)(v >> 32), CTRL, 0xf, 0xf, false);
  return ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo;
}
__device__ __forceinline__ unsigned long long readlane64(unsigned long long v, int lane) {
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(v >> 32), lane);
  return ((unsigned long long)hi << 32) | lo;
}
// acc += a * b with each real product fused into the accumulator (four FMAs,
// no separate product to keep live)
__device__ __forceinline__ void cmac(dz &acc, dz a, dz b) {
  acc.re = fma(a.re, b.re, acc.re);
  acc.re = fma(-a.im, b.im, acc.re);
  acc.im = fma(a.re, b.im, acc.im);
  acc.im = fma(a.im, b.re, acc.im);
}

// Sums over a 16-lane row of the wave, in every lane of the row, by DPP
// moves (no shared-memory traffic): lane pairs, quads, half rows, rows.
template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
  return __longlong_as_double((long long)dpp64<CTRL>((unsigned long long)__double_as_longlong(v)));
}
__device__ __forceinline__ double row16_sum(double v) {
  v = v + dpp_d<0xb1>(v);    // quad_perm [1,0,3,2]
  v = v + dpp_d<0x4e>(v);    // quad_perm [2,3,0,1]
  v = v + dpp_d<0x141>(v);   // row_half_mirror
  return v + dpp_d<0x140>(v);   // row_mirror
}
__device__ __forceinline__ dz row16_sum(dz v) { return mk(row16_sum(v.re), row16_sum(v.im)); }
// the sum over the whole wave (uniform): the four row sums added in row order
__device__ __forceinline__ double wave_sum_dpp(double v) {
  v = row16_sum(v);
  const auto rl = [](double x, int l) {
    return __longlong_as_double((long long)readlane64((unsigned long long)__double_as_longlong(x), l));
  };
  return ((rl(v, 0) + rl(v, 16)) + rl(v, 32)) + rl(v, 48);
}
__device__ __forceinline__ dz wave_sum_dpp(dz v) { return mk(wave_sum_dpp(v.re), wave_sum_dpp(v.im)); }

__device__ __forceinline__ fz operator+(fz a, fz b) { return fz{a.re + b.re, a.im + b.im}; }
__device__ __forceinline__ fz operator-(fz a, fz b) { return fz{a.re - b.re, a.im - b.im}; }
__device__ __forceinline__ fz operator*(fz a, fz b) {
  return fz{fmaf(a.re, b.re, -a.im * b.im), fmaf(a.re, b.im, a.im * b.re)};
}

// complex element traits: real type, construction, conversions to and from FP64
template <typename C> struct cx;
template <> struct cx<dz> {
  typedef double R;
  static __device__ __forceinline__ dz make(double a, double b) { return dz{a, b}; }
  static __device__ __forceinline__ dz of(dz v) { return v; }
  static __device__ __forceinline__ dz of(fz v) { return dz{v.re, v.im}; }
};
template <> struct cx<fz> {
  typedef float R;
  static __device__ __forceinline__ fz make(float a, float b) { return fz{a, b}; }
  static __device__ __forceinline__ fz of(dz v) { return fz{(float)v.re, (float)v.im}; }
  static __device__ __forceinline__ fz of(fz v) { return v; }
};
__device__ __forceinline__ dz to_dz(dz v) { return v; }
__device__ __forceinline__ dz to_dz(fz v) { return dz{v.re, v.im}; }

// Packed lattice-sum table (layout written by the host, see host.h).
namespace pk {
constexpr int E = 0, A = 1, B = 2, IA = 3, IB = 4, KXP = 5, KYP = 6, FORM = 7, MODES = 8, WS = 9, PHRE = 10, PHIM = 19,
              PROPS = 28, ROWN = 29, IMAGES = 40;
}

// Stage the packed table into LDS (all threads of the block participate).
__device__ __forceinline__ void stage_table(const double *__restrict__ pack, int len, double *lds) {
  for (int i = threadIdx.x; i < len; i += blockDim.x) lds[i] = pack[i];
  __syncthreads();
}

__device__ __forceinline__ int ufirst(int v) { return __builtin_amdgcn_readfirstlane(v); }

// integer field of the packed table (value in the low 32 bits of the slot)
__device__ __forceinline__ int pint(double slot) { return ufirst(__double2loint(slot)); }

// 1/sqrt(x) for x > 0 (finite): hardware estimate refined by one third-order
// Householder step, r <- r (1 + e/2 + 3 e^2/8) with e = 1 - x r^2.
__device__ __forceinline__ double rsqrt_pos(double x) {
  const double r = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * r, r, 1.0);
  return fma(r * e, fma(e, 0.375, 0.5), r);
}

// One series of the packed table, [K, e_0, e_1 .. e_K] (K even, coefficients of
// the highest degree first), at NC arguments: each coefficient is read once
// for all of them, the next pair while the current one is used.  Monomials by
// Horner's rule, one FMA per coefficient, or (a table whose monomials would
// round worse, see pack_pgf_table) Chebyshev coefficients by Clenshaw's
// recurrence, an addition more.
template <int NC>
__device__ __forceinline__ void series(const double *__restrict__ q, bool cheb, const double (&t)[NC], double (&f)[NC]) {
  const int K = pint(q[0]);
  const double top = q[1];
  const double *__restrict__ c = q + 2;
  double x = c[0], y = c[1];   // (K = 0: the record after this one, unused)
  if (!cheb) {
#pragma unroll
    for (int i = 0; i < NC; ++i) f[i] = top;
    // (four coefficients per pass, the pairs read in turn into two sets of registers)
#pragma unroll 1
    for (int k = 4; k <= K; k += 4) {
      const double u = c[k - 2], v = c[k - 1];
#pragma unroll
      for (int i = 0; i < NC; ++i) f[i] = fma(f[i], t[i], x);
#pragma unroll
      for (int i = 0; i < NC; ++i) f[i] = fma(f[i], t[i], y);
      x = c[k];   // (past the last pair: the next record, unused)
      y = c[k + 1];
#pragma unroll
      for (int i = 0; i < NC; ++i) f[i] = fma(f[i], t[i], u);
#pragma unroll
      for (int i = 0; i < NC; ++i) f[i] = fma(f[i], t[i], v);
    }
    if (K & 2) {
#pragma unroll
      for (int i = 0; i < NC; ++i) f[i] = fma(fma(f[i], t[i], x), t[i], y);
    }
    return;
  }
  if (K == 0) {
#pragma unroll
    for (int i = 0; i < NC; ++i) f[i] = top;
    return;
  }
  // (two arguments at a time: this form must not set the kernels' register need)
  const auto clenshaw = [&](auto width, int i0) {
    constexpr int N = decltype(width)::value;
    double b1[N], b2[N], u = x, v = y;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      b1[i] = top;
      b2[i] = 0.0;
    }
    const auto step = [&](double ck) {
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const double n = fma(t[i0 + i] + t[i0 + i], b1[i], ck - b2[i]);
        b2[i] = b1[i];
        b1[i] = n;
      }
    };
#pragma unroll 1
    for (int k = 2;; k += 2) {   // the pair (u, v) = (c_j, c_{j-1}); the last v is c_0
      step(u);
      if (k >= K) break;
      step(v);
      u = c[k];
      v = c[k + 1];
    }
#pragma unroll
    for (int i = 0; i < N; ++i) f[i0 + i] = fma(t[i0 + i], b1[i], v - b2[i]);
  };
#pragma unroll
  for (int i = 0; i + 1 < NC; i += 2) clenshaw(std::integral_constant<int, 2>(), i);
  if (NC & 1) clenshaw(std::integral_constant<int, 1>(), NC - 1);
}

// Two series of one degree at the same arguments, [K, 0, (s_0, d_0) .. (s_K, d_K)]:
// one read gives a coefficient of both.
template <int W>
__device__ __forceinline__ void series_pair(const double *__restrict__ q, bool cheb, const double (&t)[W], double (&s)[W],
                                            double (&d)[W]) {
  const int K = pint(q[0]);
  const double *__restrict__ c = q + 2;
  if (!cheb) {
    double x = c[0], y = c[1];
#pragma unroll
    for (int w = 0; w < W; ++w) {
      s[w] = x;
      d[w] = y;
    }
    x = c[2];   // (K = 0: the next record, unused)
    y = c[3];
#pragma unroll 1
    for (int k = 2; k <= K; k += 2) {
      const double u = c[2 * k], v = c[2 * k + 1];
#pragma unroll
      for (int w = 0; w < W; ++w) {
        s[w] = fma(s[w], t[w], x);
        d[w] = fma(d[w], t[w], y);
      }
      x = c[2 * k + 2];
      y = c[2 * k + 3];
#pragma unroll
      for (int w = 0; w < W; ++w) {
        s[w] = fma(s[w], t[w], u);
        d[w] = fma(d[w], t[w], v);
      }
    }
    return;
  }
#pragma unroll 1
  for (int h = 0; h < 2; ++h) {   // Clenshaw, one series after the other
    double b1[W], b2[W], f[W];
#pragma unroll
    for (int w = 0; w < W; ++w) b1[w] = b2[w] = 0.0;
#pragma unroll 1
    for (int k = 0; k < K; ++k) {
      const double ck = c[2 * k + h];
#pragma unroll
      for (int w = 0; w < W; ++w) {
        const double n = fma(t[w] + t[w], b1[w], ck - b2[w]);
        b2[w] = b1[w];
        b1[w] = n;
      }
    }
    const double last = c[2 * K + h];
#pragma unroll
    for (int w = 0; w < W; ++w) {
      f[w] = fma(t[w], b1[w], last - b2[w]);
      if (h) d[w] = f[w];
      else s[w] = f[w];
    }
  }
}

// the next record after a series at offset `off`
__device__ __forceinline__ int after_series(const double *__restrict__ P, int off) { return off + 2 + pint(P[off]); }

// The NS images (+-m, +-n) of one record at W separations: f(t) / R (or, for a
// touching image, E times the H series), added to the spatial sum with the
// image phases.  Images (s m, s n) and (-s m, -s n) have conjugate phases.
template <bool TOUCH, int W, int NS>
__device__ __forceinline__ void image_group(const double *__restrict__ R, bool cheb, double E, const double (&R2)[NS * W],
                                            const bool (&touch)[TOUCH ? NS * W : 1], double (&sre)[W], double (&sim)[W]) {
  double t[NS * W], sc[NS * W], f[NS * W];
#pragma unroll
  for (int i = 0; i < NS * W; ++i) {
    double Rw;
    if (TOUCH) {   // a touching image can sit at R = 0 (its H series is evaluated at x = 0)
      sc[i] = rsqrt(R2[i]);
      Rw = R2[i] > 0.0 ? R2[i] * sc[i] : 0.0;
    } else {       // separations of non-touching elements never vanish
      sc[i] = rsqrt_pos(R2[i]);
      Rw = R2[i] * sc[i];
    }
    t[i] = fma(Rw, R[0], R[1]);   // the fit's argument
  }
  series<NS * W>(R + 6, cheb, t, f);
  if (TOUCH) {
    bool any = false;
#pragma unroll
    for (int i = 0; i < NS * W; ++i) any = any || touch[i];
    if (any) {
      double h[NS * W];
      series<NS * W>(R + after_series(R, 6), cheb, t, h);
#pragma unroll
      for (int i = 0; i < NS * W; ++i)
        if (touch[i]) {
          f[i] = h[i];
          sc[i] = E;
        }
    }
  }
#pragma unroll
  for (int s = 0; s < NS; s += 2) {
    const double cre = R[2 + s], cim = R[3 + s];
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const double g = f[s * W + w] * sc[s * W + w];
      if (NS == 1) {
        sre[w] = fma(cre, g, sre[w]);
      } else {
        const double g2 = f[(s + 1) * W + w] * sc[(s + 1) * W + w];
        sre[w] = fma(cre, g + g2, sre[w]);
        sim[w] = fma(cim, g - g2, sim[w]);
      }
    }
  }
}

// g_p at W separations d[w] = r - r'_w at once (one test point, W source
// points), from the packed table P.
//
// Images: (+-m, +-n) lie in the same range of R and share one series, so the
// record's coefficients are read once for the up to 4 W arguments, which is
// what keeps the LDS reads (one per coefficient and wave) below the FMAs.
// Orders: with the terms K_pq real (the imaginary parts of the propagating
// orders apart), sum_q K_pq e^{-j 2 pi q dy/b} = K_p0 + sum_{q>0} (S_q cos -
// j D_q sin), S and D the sums and differences of the series of (p, q) and
// (p, -q), and the rows p are summed by Horner's rule in e^{-j 2 pi dx/a}.
// An FP64 FMA issues every four cycles per SIMD, and this is bound by them.
//
// When TOUCH is true, `mask` lists the lattice images (bit (m+1)*3 + (n+1))
// whose 1/(4 pi R) part is integrated in closed form elsewhere; for those
// images the remainder H(x) E/(4 pi) is used, so the value returned is
// g_p - sum_touching e^{j kt.rho}/(4 pi R).
//
// REV (non-touching separations only): also g_p at -d[w] into rev[w].  For a
// real wavenumber every spatial image term is a real function of R times the
// image phase e^{j kt.rho_mn}, and the images (m, n), (-m, -n) share that
// function, so the spatial sum at -d is the conjugate of the one at d.  A
// spectral term e^{-j k_tpq.Delta} K_pq(z) has K_pq even in z and real for an
// evanescent order, so it too conjugates, except for the propagating orders,
// whose K_pq is complex.  Hence
//   g_p(-d) = conj(g_p(d)) + conj(ph0) 2j sum_{propagating} conj(e^{-j k_tpq.Delta}) Im K_pq(z),
// with ph0 the phase of the nearest-image shift (which flips with d).
template <bool TOUCH, int W, bool REV = false>
__device__ __forceinline__ void pgf_eval_w(const double *__restrict__ P, const double (&d)[W][3], int mask,
                                           dz (&out)[W], dz *rev = nullptr) {
  const double a = P[pk::A], b = P[pk::B], E = P[pk::E];
  const bool cheb = pint(P[pk::FORM]) != 0;
  double dx[W], dy[W], dz2[W], sre[W], sim[W];
  int im0[W], in0[W];
#pragma unroll
  for (int w = 0; w < W; ++w) {
    const double m0 = rint(d[w][0] * P[pk::IA]), n0 = rint(d[w][1] * P[pk::IB]);
    dx[w] = fma(-m0, a, d[w][0]);
    dy[w] = fma(-n0, b, d[w][1]);
    dz2[w] = d[w][2] * d[w][2];
    im0[w] = (int)m0;
    in0[w] = (int)n0;
    sre[w] = 0.0;
    sim[w] = 0.0;
  }
  // spatial series: rows m = 0, 1, ... of the records n = 0 .. P[ROWN + m] - 1
  int off = pk::IMAGES;
#pragma unroll 1
  for (int m = 0; m <= kPgfM; ++m) {
    const int nn = pint(P[pk::ROWN + m]);
    double xp[W], xm[W];   // (dx +- m a)^2 + dz^2
    const double ma = (double)m * a;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const double X = dx[w] + ma, Y = dx[w] - ma;
      xp[w] = fma(X, X, dz2[w]);
      xm[w] = fma(Y, Y, dz2[w]);
    }
    const auto touching = [&](int w, int sm, int sn) {   // image (sm, sn) of the wrapped separation
      const int um = sm - im0[w], un = sn - in0[w];
      return um >= -1 && um <= 1 && un >= -1 && un <= 1 && ((mask >> ((um + 1) * 3 + (un + 1))) & 1);
    };
#pragma unroll 1
    for (int n = 0; n < nn; ++n) {
      const double *R = P + off;
      const double nb = (double)n * b;
      off += ufirst(__double2hiint(R[6]));   // the record's length
      const bool fit = TOUCH && m <= 1 && n <= 1;   // the records with an H series
      if (m > 0 && n > 0) {
        double R2[4 * W];
        bool tc[TOUCH ? 4 * W : 1] = {};
#pragma unroll
        for (int w = 0; w < W; ++w) {
          const double yp = dy[w] + nb, ym = dy[w] - nb;
          R2[w] = fma(yp, yp, xp[w]);
          R2[W + w] = fma(ym, ym, xm[w]);
          R2[2 * W + w] = fma(ym, ym, xp[w]);
          R2[3 * W + w] = fma(yp, yp, xm[w]);
          if (fit) {
            tc[w] = touching(w, m, n);
            tc[TOUCH ? W + w : 0] = touching(w, -m, -n);
            tc[TOUCH ? 2 * W + w : 0] = touching(w, m, -n);
            tc[TOUCH ? 3 * W + w : 0] = touching(w, -m, n);
          }
        }
        image_group<TOUCH, W, 4>(R, cheb, E, R2, tc, sre, sim);
      } else if (m > 0 || n > 0) {
        double R2[2 * W];
        bool tc[TOUCH ? 2 * W : 1] = {};
#pragma unroll
        for (int w = 0; w < W; ++w) {
          const double yp = dy[w] + nb, ym = dy[w] - nb;
          R2[w] = fma(yp, yp, xp[w]);
          R2[W + w] = fma(ym, ym, xm[w]);
          if (fit) {
            tc[w] = touching(w, m, n);
            tc[TOUCH ? W + w : 0] = touching(w, -m, -n);
          }
        }
        image_group<TOUCH, W, 2>(R, cheb, E, R2, tc, sre, sim);
      } else {
        double R2[W];
        bool tc[TOUCH ? W : 1] = {};
#pragma unroll
        for (int w = 0; w < W; ++w) {
          R2[w] = fma(dy[w], dy[w], xp[w]);
          if (fit) tc[w] = touching(w, 0, 0);
        }
        image_group<TOUCH, W, 1>(R, cheb, E, R2, tc, sre, sim);
      }
    }
  }

  // spectral series in w = (z E)^2
  double tw[W];
  dz bx[W], by[W], acc[W];
#pragma unroll
  for (int w = 0; w < W; ++w) {
    tw[w] = fma(dz2[w], P[pk::WS], -1.0);
    double s1, c1;
    sincospi(-2.0 * dx[w] * P[pk::IA], &s1, &c1);
    bx[w] = mk(c1, s1);
    sincospi(-2.0 * dy[w] * P[pk::IB], &s1, &c1);
    by[w] = mk(c1, s1);
    acc[w] = mk(0.0, 0.0);
  }
  off = pint(P[pk::MODES]);
  const int hd = ufirst(__double2hiint(P[pk::MODES]));   // rows p = plo .. phi: plo + 8 | (phi + 8) << 8
  const int plo = (hd & 0xff) - 8, phi = (hd >> 8) - 8;
#pragma unroll 1
  for (int p = phi; p >= plo; --p) {
    const int nq = pint(P[off]);
    const bool odd = ufirst(__double2hiint(P[off])) != 0;   // the row has differences
    off += 2;
    double k0[W];
    series<W>(P + off, cheb, tw, k0);
    off = after_series(P, off);
#pragma unroll
    for (int w = 0; w < W; ++w)
      acc[w] = mk(fma(acc[w].re, bx[w].re, fma(-acc[w].im, bx[w].im, k0[w])), fma(acc[w].re, bx[w].im, acc[w].im * bx[w].re));
    dz e[W];
#pragma unroll
    for (int w = 0; w < W; ++w) e[w] = by[w];
#pragma unroll 1
    for (int q = 1; q <= nq; ++q) {
      if (odd) {
        double s[W], d[W];
        series_pair<W>(P + off, cheb, tw, s, d);
        off += 2 + 2 * (pint(P[off]) + 1);
#pragma unroll
        for (int w = 0; w < W; ++w) {
          acc[w].re = fma(s[w], e[w].re, acc[w].re);
          acc[w].im = fma(d[w], e[w].im, acc[w].im);
        }
      } else {
        double s[W];
        series<W>(P + off, cheb, tw, s);
        off = after_series(P, off);
#pragma unroll
        for (int w = 0; w < W; ++w) acc[w].re = fma(s[w], e[w].re, acc[w].re);
      }
#pragma unroll
      for (int w = 0; w < W; ++w) e[w] = e[w] * by[w];
    }
  }
  // times bx^plo (plo <= 0)
#pragma unroll 1
  for (int p = plo; p < 0; ++p) {
#pragma unroll
    for (int w = 0; w < W; ++w) acc[w] = acc[w] * conjz(bx[w]);
  }
  // propagating orders: e^{-j k_pq Delta} j Im K_pq
  double pr[W], pi[W];
#pragma unroll
  for (int w = 0; w < W; ++w) pr[w] = pi[w] = 0.0;
  off = pint(P[pk::PROPS]);
  const int np = ufirst(__double2hiint(P[pk::PROPS]));
#pragma unroll 1
  for (int i = 0; i < np; ++i) {
    const int p = pint(P[off]), q = ufirst(__double2hiint(P[off]));
    off += 2;
    double ki[W];
    series<W>(P + off, cheb, tw, ki);
    off = after_series(P, off);
    dz e[W];
#pragma unroll
    for (int w = 0; w < W; ++w) e[w] = mk(1.0, 0.0);
#pragma unroll 1
    for (int j = 0; j < (p < 0 ? -p : p); ++j) {
#pragma unroll
      for (int w = 0; w < W; ++w) e[w] = e[w] * (p < 0 ? conjz(bx[w]) : bx[w]);
    }
#pragma unroll 1
    for (int j = 0; j < (q < 0 ? -q : q); ++j) {
#pragma unroll
      for (int w = 0; w < W; ++w) e[w] = e[w] * (q < 0 ? conjz(by[w]) : by[w]);
    }
#pragma unroll
    for (int w = 0; w < W; ++w) {
      pr[w] = fma(e[w].re, ki[w], pr[w]);
      pi[w] = fma(e[w].im, ki[w], pi[w]);
    }
  }
  const bool kt0 = P[pk::KXP] == 0.0 && P[pk::KYP] == 0.0;   // normal incidence: e^{-j kt.Delta} = 1
#pragma unroll
  for (int w = 0; w < W; ++w) {
    dz u = mk(1.0, 0.0);
    if (!kt0) {
      double s1, c1;
      sincospi(-fma(P[pk::KXP], dx[w], P[pk::KYP] * dy[w]), &s1, &c1);
      u = mk(c1, s1);
    }
    const dz k = u * mk(acc[w].re - pi[w], acc[w].im + pr[w]);
    const int i0 = (im0[w] + 1) * 3 + (in0[w] + 1);
    const dz ph = mk(P[pk::PHRE + i0], P[pk::PHIM + i0]);
    out[w] = ph * mk(sre[w] + k.re, sim[w] + k.im);
    if (REV) {
      const dz c = conjz(u) * mk(pr[w], -pi[w]);   // conj(e^{-j k_pq Delta}) Im K_pq, summed
      rev[w] = conjz(out[w]) + conjz(ph) * mk(-2.0 * c.im, 2.0 * c.re);
    }
  }
}

// single separation
template <bool TOUCH>
__device__ __forceinline__ dz pgf_eval(const double *__restrict__ P, double dx, double dy, double dzv, int mask) {
  const double d[1][3] = {{dx, dy, dzv}};
  dz o[1];
  pgf_eval_w<TOUCH, 1>(P, d, mask, o);
  return o[0];
}

// ---------------------------------------------------------------- potentials
__device__ __forceinline__ void sub3(const double *a, const double *b, double *o) {
  o[0] = a[0] - b[0];
  o[1] = a[1] - b[1];
  o[2] = a[2] - b[2];
}
__device__ __forceinline__ double dot3(const double *a, const double *b) {
  return fma(a[0], b[0], fma(a[1], b[1], a[2] * b[2]));
}
__device__ __forceinline__ void cross3(const double *a, const double *b, double *o) {
  o[0] = a[1] * b[2] - a[2] * b[1];
  o[1] = a[2] * b[0] - a[0] * b[2];
  o[2] = a[0] * b[1] - a[1] * b[0];
}
__device__ __forceinline__ void unit3(double *v) {
  const double s = rsqrt(dot3(v, v));
  v[0] *= s;
  v[1] *= s;
  v[2] *= s;
}

// Integrals of 1/|r - r'| and |r - r'| over the flat triangle (A, B, C) for the
// observation point r (polygon formulas: edge logarithms and angle terms).
__device__ inline void tri_potentials(const double *A, const double *B, const double *C, const double *r,
                                      double &iinv, double &ione) {
  const double *V[3] = {A, B, C};
  double e1[3], e2[3], nrm[3];
  sub3(B, A, e1);
  sub3(C, A, e2);
  cross3(e1, e2, nrm);
  unit3(nrm);
  double ra[3];
  sub3(r, A, ra);
  const double d = dot3(ra, nrm), ad = fabs(d);
  const double rho0[3] = {r[0] - d * nrm[0], r[1] - d * nrm[1], r[2] - d * nrm[2]};
  double sinv = 0.0, sedge = 0.0;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const double *Pm = V[i], *Pp = V[(i + 1) % 3], *Po = V[(i + 2) % 3];
    double l[3], w[3], u[3], tmp[3];
    sub3(Pp, Pm, l);
    unit3(l);
    sub3(Pm, Po, w);
    const double wl = dot3(w, l);
    u[0] = w[0] - wl * l[0];
    u[1] = w[1] - wl * l[1];
    u[2] = w[2] - wl * l[2];
    unit3(u);
    sub3(Pm, rho0, tmp);
    const double t = dot3(tmp, u);
    double pp[3], pm[3];
    sub3(Pp, r, pp);
    sub3(Pm, r, pm);
    const double lp = dot3(pp, l), lm = dot3(pm, l);
    const double Rp = sqrt(dot3(pp, pp)), Rm = sqrt(dot3(pm, pm));
    const double R02 = fma(t, t, d * d);
    double f = 0.0;
    if (t != 0.0) {
      const bool neg = lp < 0.0 && lm < 0.0;
      const double num = neg ? Rm - lm : Rp + lp;
      const double den = neg ? Rp - lp : Rm + lm;
      if (num > 0.0 && den > 0.0) f = log(num / den);
    }
    const double beta = atan2(t * lp, fma(ad, Rp, R02)) - atan2(t * lm, fma(ad, Rm, R02));
    sinv += t * f - ad * beta;
    sedge += t * (fma(R02, f, lp * Rp) - lm * Rm);
  }
  iinv = sinv;
  ione = (d * d * sinv + 0.5 * sedge) / 3.0;
}

// Face f's part of the integrals of 1/|r - r'| (P) and (r' - r)/|r - r'| (V1)
// over the tetrahedron with vertices v[4][3] (divergence theorem): summed over
// the four faces they are the integrals.
__device__ inline void tet_potentials_face(const double (*v)[3], int f, const double *r, double &P, double *V1) {
  // faces 123, 032, 013, 021
  const double *A = v[f == 0 ? 1 : 0], *B = v[f == 0 || f == 3 ? 2 : (f == 1 ? 3 : 1)],
               *C = v[f == 0 || f == 2 ? 3 : (f == 1 ? 2 : 1)];
  double c[3], e1[3], e2[3], n[3], ac[3];
  for (int d = 0; d < 3; ++d) c[d] = 0.25 * (v[0][d] + v[1][d] + v[2][d] + v[3][d]);
  sub3(B, A, e1);
  sub3(C, A, e2);
  cross3(e1, e2, n);
  unit3(n);
  sub3(A, c, ac);
  if (dot3(ac, n) < 0.0) {
    n[0] = -n[0];
    n[1] = -n[1];
    n[2] = -n[2];
  }
  double iinv, ione;
  tri_potentials(A, B, C, r, iinv, ione);
  double ar[3];
  sub3(A, r, ar);
  P = 0.5 * dot3(ar, n) * iinv;
  for (int d = 0; d < 3; ++d) V1[d] = ione * n[d];
}

// touching-image mask of two vertex sets (canonical ids + packed offsets)
__device__ __forceinline__ int touch_mask(const int32_t *ct, const int32_t *ot, int nt_, const int32_t *cs,
                                          const int32_t *os, int ns) {
  int mask = 0;
  for (int i = 0; i < nt_; ++i)
    for (int j = 0; j < ns; ++j)
      if (ct[i] == cs[j]) {
        const int dm = (os[j] & 15) - (ot[i] & 15), dn = (os[j] >> 4) - (ot[i] >> 4);
        mask |= 1 << ((dm + 1) * 3 + (dn + 1));
      }
  return mask;
}

}  // namespace vie
