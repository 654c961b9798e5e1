// Far element pairs of the mixed-precision operator (FP32 entries).
//
// Every contribution is added to its FP32 entry in FP64 and rounded, so a
// contribution that moves by a few 1e-16 moves isolated entries to the
// neighbouring FP32 value: 1e-7 of them, which leaves Z x within 3e-11 and the
// solution within 1e-9 in norm, but a single component of it 1e-7 off (N =
// 37,376).  A path that solves to 1e-12 should not move by that with the form
// of a series, so the arithmetic of these contributions is held fixed, to the
// bit: the terms come from one evaluation (PgfTerms::fixed), each as
// its Chebyshev series by Clenshaw's recurrence; images and orders are summed
// in the order of their grids, and the point pairs of an element pair one
// after another by one lane.  k_fill.hip, whose entries are FP64, is free of
// this and takes whichever form is fastest; touching pairs are FP64 in both
// paths and come from there.
#include "fill.h"

namespace vie {

// Packed table of these kernels (pack_pgf_fixed): header, per-order offsets,
// image records, order records.
namespace pkf {
constexpr int E = 0, A = 1, B = 2, IA = 3, IB = 4, KX = 5, KY = 6, TPA = 7, TPB = 8, WS = 9, PHRE = 10, PHIM = 19,
              NIMG = 28, MODES = 32, ROWS = 116, IMAGES = 128;
}

// W Chebyshev series with the same coefficients c[0..K] (K even, zero-padded)
// at W arguments t[w]: interleaved Clenshaw recurrences, two coefficients per
// step, each coefficient read once for all W.
template <int W>
__device__ __forceinline__ void clenshaw_w(const double *__restrict__ c, int K, const double (&t)[W], double (&f)[W]) {
  double b1[W], b2[W], t2[W];
#pragma unroll
  for (int w = 0; w < W; ++w) {
    b1[w] = b2[w] = 0.0;
    t2[w] = t[w] + t[w];
  }
  // four coefficients per pass, all read before the first is used, so one
  // read's latency is exposed per four coefficients rather than per two
  const auto pair = [&](double ck, double ck1) {
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const double bk = fma(t2[w], b1[w], ck - b2[w]);
      const double bk1 = fma(t2[w], bk, ck1 - b1[w]);
      b2[w] = bk;
      b1[w] = bk1;
    }
  };
  int k = K;
#pragma unroll 1
  for (; k >= 8; k -= 8) {
    const double c0 = c[k], c1 = c[k - 1], c2 = c[k - 2], c3 = c[k - 3];
    const double c4 = c[k - 4], c5 = c[k - 5], c6 = c[k - 6], c7 = c[k - 7];
    pair(c0, c1);
    pair(c2, c3);
    pair(c4, c5);
    pair(c6, c7);
  }
  if (k >= 4) {   // (K is a multiple of 4: what remains is 4 or 0)
    const double c0 = c[k], c1 = c[k - 1], c2 = c[k - 2], c3 = c[k - 3];
    pair(c0, c1);
    pair(c2, c3);
    k -= 4;
  }
#pragma unroll 1
  for (; k >= 2; k -= 2) pair(c[k], c[k - 1]);
#pragma unroll
  for (int w = 0; w < W; ++w) f[w] = fma(t[w], b1[w], c[0] - b2[w]);
}

// g_p at W separations d[w] = r - r'_w of non-touching elements (one point
// against W), from the packed table P.  The table entries are read once for
// all W separations and the W Clenshaw recurrences run interleaved.
// REV: also g_p at -d[w] into rev[w] (see pgf_eval_w).
template <int W, bool REV = false>
__device__ __forceinline__ void pgf_fixed_w(const double *__restrict__ P, const double (&d)[W][3], dz (&out)[W],
                                            dz *rev = nullptr) {
  const double a = P[pkf::A], b = P[pkf::B], E = P[pkf::E];
  double dx[W], dy[W], dz2[W], sre[W], sim[W];
  int im0[W], in0[W];
#pragma unroll
  for (int w = 0; w < W; ++w) {
    const double m0 = rint(d[w][0] * P[pkf::IA]), n0 = rint(d[w][1] * P[pkf::IB]);
    dx[w] = fma(-m0, a, d[w][0]);
    dy[w] = fma(-n0, b, d[w][1]);
    dz2[w] = d[w][2] * d[w][2];
    im0[w] = (int)m0;
    in0[w] = (int)n0;
    sre[w] = 0.0;
    sim[w] = 0.0;
  }
  // spatial series
  const int nimg = pint(P[pkf::NIMG]);
  int off = pkf::IMAGES;
#pragma unroll 1
  for (int i = 0; i < nimg; ++i) {
    const double *R = P + off;
    const double ts = R[0], t0 = R[1], cre = R[2], cim = R[3];   // t = ts R + t0
    const int im = pint(R[4]), in = pint(R[5]), K = pint(R[6]);
    off += pint(R[7]);
    double t[W], sc[W];
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const double X = fma((double)im, a, dx[w]), Y = fma((double)in, b, dy[w]);
      const double R2 = fma(X, X, fma(Y, Y, dz2[w]));
      const double rinv = rsqrt_pos(R2), Rw = R2 * rinv;
      t[w] = fma(Rw, ts, t0);
      sc[w] = rinv;
    }
    // W interleaved Clenshaw recurrences on the F coefficients
    double b1[W], b2[W];
#pragma unroll
    for (int w = 0; w < W; ++w) b1[w] = b2[w] = 0.0;
    const double *c = R + 8;
    // four coefficients per pass, read before the first is used (as in clenshaw_w)
    double t2[W];
#pragma unroll
    for (int w = 0; w < W; ++w) t2[w] = t[w] + t[w];
    const auto pair = [&](double ck, double ck1) {
#pragma unroll
      for (int w = 0; w < W; ++w) {
        const double bk = fma(t2[w], b1[w], ck - b2[w]);
        const double bk1 = fma(t2[w], bk, ck1 - b1[w]);
        b2[w] = bk;
        b1[w] = bk1;
      }
    };
    int k = K;
#pragma unroll 1
    for (; k >= 8; k -= 8) {
      const double c0 = c[k], c1 = c[k - 1], c2 = c[k - 2], c3 = c[k - 3];
      const double c4 = c[k - 4], c5 = c[k - 5], c6 = c[k - 6], c7 = c[k - 7];
      pair(c0, c1);
      pair(c2, c3);
      pair(c4, c5);
      pair(c6, c7);
    }
    if (k >= 4) {   // (K is a multiple of 4: what remains is 4 or 0)
      const double c0 = c[k], c1 = c[k - 1], c2 = c[k - 2], c3 = c[k - 3];
      pair(c0, c1);
      pair(c2, c3);
      k -= 4;
    }
#pragma unroll 1
    for (; k >= 2; k -= 2) pair(c[k], c[k - 1]);
    double f[W];
#pragma unroll
    for (int w = 0; w < W; ++w) f[w] = fma(t[w], b1[w], c[0] - b2[w]);
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const double g = f[w] * sc[w];
      sre[w] = fma(cre, g, sre[w]);
      sim[w] = fma(cim, g, sim[w]);
    }
  }

  // spectral series: the W separations share every mode's coefficient reads
  // and run W interleaved Clenshaw recurrences in w = (z E)^2; the Floquet
  // phases e^{-j k_tpq . Delta_t} of each separation by recurrence in p and q
  double tw[W], kre[W], kim[W], cre_[W], cim_[W];
  dz erow[W], bx[W], by[W];   // erow: phase of (p, q = -4); steps in p and in q
  const bool kt0 = P[pkf::KX] == 0.0 && P[pkf::KY] == 0.0;   // normal incidence: e^{-j kt.Delta} = 1
#pragma unroll
  for (int w = 0; w < W; ++w) {
    tw[w] = fma(dz2[w] * E * E, P[pkf::WS], -1.0);
    double s0, c0, s1, c1;
    sincos(-P[pkf::TPA] * dx[w], &s1, &c1);
    bx[w] = mk(c1, s1);
    sincos(-P[pkf::TPB] * dy[w], &s1, &c1);
    by[w] = mk(c1, s1);
    const dz bx4 = conjz(bx[w] * bx[w] * bx[w] * bx[w]), by4 = conjz(by[w] * by[w] * by[w] * by[w]);
    if (kt0) {
      erow[w] = bx4 * by4;   // (p, q) = (-4, -4)
    } else {
      sincos(-P[pkf::KX] * dx[w], &s0, &c0);
      const dz ex = mk(c0, s0) * bx4;   // p = -4
      sincos(-P[pkf::KY] * dy[w], &s0, &c0);
      erow[w] = ex * (mk(c0, s0) * by4);
    }
    kre[w] = 0.0;
    kim[w] = 0.0;
    cre_[w] = 0.0;
    cim_[w] = 0.0;
  }
  // rows of the grid: only the slots from the row's first to its last mode
  // (the phases of the slots below reached by the same products as before)
#pragma unroll 1
  for (int p = 0; p < kPgfSide; ++p) {
    const int rr = pint(P[pkf::ROWS + p]);
    const int qlo = rr & 0xff, qend = rr >> 8;
    dz e[W];
#pragma unroll
    for (int w = 0; w < W; ++w) e[w] = erow[w];
#pragma unroll 1
    for (int q = 0; q < qlo; ++q) {
#pragma unroll
      for (int w = 0; w < W; ++w) e[w] = e[w] * by[w];
    }
#pragma unroll 1
    for (int q = qlo; q < qend; ++q) {
      const double slot = P[pkf::MODES + p * kPgfSide + q];
      const int moff = pint(slot);
      if (moff > 0) {
        const double *M = P + moff;
        const int kc = ufirst(__double2hiint(slot));   // K | cplx << 16
        const int K = kc & 0xffff;
        double kr[W];
        clenshaw_w<W>(M + 4, K, tw, kr);
        if ((kc >> 16) != 0) {
          double ki[W];
          clenshaw_w<W>(M + 4 + K + 4, K, tw, ki);
#pragma unroll
          for (int w = 0; w < W; ++w) {
            kre[w] += e[w].re * kr[w] - e[w].im * ki[w];
            kim[w] += e[w].re * ki[w] + e[w].im * kr[w];
            if (REV) {   // conj(e) Im K_pq of a propagating order
              cre_[w] = fma(e[w].re, ki[w], cre_[w]);
              cim_[w] = fma(-e[w].im, ki[w], cim_[w]);
            }
          }
        } else {
#pragma unroll
          for (int w = 0; w < W; ++w) {
            kre[w] = fma(e[w].re, kr[w], kre[w]);
            kim[w] = fma(e[w].im, kr[w], kim[w]);
          }
        }
      }
#pragma unroll
      for (int w = 0; w < W; ++w) e[w] = e[w] * by[w];
    }
#pragma unroll
    for (int w = 0; w < W; ++w) erow[w] = erow[w] * bx[w];
  }
#pragma unroll
  for (int w = 0; w < W; ++w) {
    const int pi = (im0[w] + 1) * 3 + (in0[w] + 1);
    const dz ph = mk(P[pkf::PHRE + pi], P[pkf::PHIM + pi]);
    out[w] = ph * mk(sre[w] + kre[w], sim[w] + kim[w]);
    if (REV) rev[w] = conjz(out[w]) + conjz(ph) * mk(-2.0 * cim_[w], 2.0 * cre_[w]);
  }
}

// Scatter the 16 face-pair contributions of tet pair (T, S) into Z (TRANS:
// entry (m, n) goes to (n, m) of the output).
template <bool TRANS = false>
__device__ __forceinline__ void scatter_tt(const Moments &M, const TetGeom &gt, const TetGeom &gs,
                                           const TetFace *__restrict__ t2f, int T, int S,
                                           const dz *__restrict__ alpha, const dz *__restrict__ gsrc,
                                           const dz *__restrict__ kappa, double k0sq9, const ZOut &out,
                                           bool near) {
  const dz ks = kappa[S];
  double qv[4][3];
  dz bl[4];
  int64_t col[4];
  for (int l = 0; l < 4; ++l) {
    for (int d = 0; d < 3; ++d) qv[l][d] = gs.v[l][d] - gs.c[d];
    bl[l] = gsrc[4 * S + l] * ks;
    col[l] = t2f[4 * S + l].unknown;
  }
  for (int k = 0; k < 4; ++k) {
    double pk[3];
    for (int d = 0; d < 3; ++d) pk[d] = gt.v[k][d] - gt.c[d];
    // muv - p~.mv
    dz base = M.muv;
    for (int d = 0; d < 3; ++d) base = base - pk[d] * M.mv[d];
    const dz ak = alpha[4 * T + k];
    const int64_t row = t2f[4 * T + k].unknown;
    for (int l = 0; l < 4; ++l) {
      dz I = base;
      for (int d = 0; d < 3; ++d) I = I - qv[l][d] * M.mu[d];
      I = I + dot3(pk, qv[l]) * M.m0;
      const dz v = M.m0 - k0sq9 * I;
      if (TRANS) zput(out, col[l], row, (ak * bl[l]) * v, near);
      else zput(out, row, col[l], (ak * bl[l]) * v, near);
    }
  }
}

// Far tet pairs: 4 x 4 product rule.  One wave = one test tet x 64 source tets.
// sym > 0 writes the swapped pair's block (S, T) too, from the pair's own
// moments at normal incidence, else (REV) from those of the reversed
// separations, which are summed per lane in LDS (16 doubles after the table,
// one column per thread), not in registers, so that the kernel keeps two waves
// per SIMD without spilling.
template <bool REV>
__device__ __forceinline__ void tt_far_c_body(const double *__restrict__ pack, int packlen,
                                              const QuadRules *__restrict__ qr, const TetGeom *__restrict__ tg,
                                              const TetFace *__restrict__ t2f, const int32_t *__restrict__ test_list,
                                              int ntest, const int32_t *__restrict__ src_list, int nsrc,
                                              const dz *__restrict__ alpha, const dz *__restrict__ gsrc,
                                              const dz *__restrict__ kappa, double k0sq9, const ZOut &out,
                                              const ZOut &outT, int sym, int bx_, int by_) {
  extern __shared__ double s_tab[];
  // one list against itself: a block whose source positions all lie at or
  // below its test positions has nothing to do (the whole block returns)
  if (sym == 2 && bx_ * 64 + 63 <= by_ * 4) return;
  stage_table(pack, packlen, s_tab);
  const double *__restrict__ P = s_tab;
  double *__restrict__ mr = s_tab + ((packlen + 1) & ~1) + threadIdx.x;   // REV: entry e at mr[256 e]

  const int ti = uniform(by_ * 4 + (threadIdx.x >> 6));
  const int si = bx_ * 64 + (threadIdx.x & 63);
  if (ti >= ntest || si >= nsrc) return;
  if (sym == 2 && si <= ti) return;
  const int T = uniform(test_list[ti]);
  const int S = src_list[si];
  const TetGeom &gt = tg[T];
  double wq;
  double up[4][3], dc[3];
  {
    const TetGeom gs = tg[S];
    if (touch_mask(gt.canon, gt.off, 4, gs.canon, gs.off, 4)) return;  // touching pairs: k_tt_near
    wq = 0.25 * gs.vol;
    for (int d = 0; d < 3; ++d) dc[d] = gt.c[d] - gs.c[d];
    // source points relative to the source centroid
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        double s = 0;
        for (int k = 0; k < 4; ++k) s = fma(qr->tet4[j][k], gs.v[k][d], s);
        up[j][d] = s - gs.c[d];
      }
  }
  const double wt = 0.25 * gt.vol;
  Moments M;
  moments_zero(M);
  if (REV)
    for (int e = 0; e < 16; ++e) mr[256 * e] = 0.0;
  // one test point against the four source points per lattice-sum call
#pragma unroll 1
  for (int i = 0; i < 4; ++i) {
    double u[3];
    for (int d = 0; d < 3; ++d) {
      double s = 0;
      for (int k = 0; k < 4; ++k) s = fma(qr->tet4[i][k], gt.v[k][d], s);
      u[d] = s - gt.c[d];
    }
    double sep[4][3];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int d = 0; d < 3; ++d) sep[j][d] = dc[d] + u[d] - up[j][d];
    dz g[4], gr[REV ? 4 : 1];
    pgf_fixed_w<4, REV>(P, sep, g, gr);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const dz gw = (wt * wq) * g[j];
      M.m0 = M.m0 + gw;
      for (int d = 0; d < 3; ++d) {
        axpy(M.mu[d], u[d], gw);
        axpy(M.mv[d], up[j][d], gw);
      }
      axpy(M.muv, dot3(u, up[j]), gw);
    }
    if (REV) {
      // swapped pair (S, T): its test offsets are up_j, its source offsets u
      Moments R;
      moments_zero(R);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const dz grw = (wt * wq) * gr[j];
        R.m0 = R.m0 + grw;
        for (int d = 0; d < 3; ++d) {
          axpy(R.mu[d], up[j][d], grw);
          axpy(R.mv[d], u[d], grw);
        }
        axpy(R.muv, dot3(u, up[j]), grw);
      }
      mr[0] += R.m0.re;
      mr[256] += R.m0.im;
      for (int d = 0; d < 3; ++d) {
        mr[256 * (2 + 2 * d)] += R.mu[d].re;
        mr[256 * (3 + 2 * d)] += R.mu[d].im;
        mr[256 * (8 + 2 * d)] += R.mv[d].re;
        mr[256 * (9 + 2 * d)] += R.mv[d].im;
      }
      mr[256 * 14] += R.muv.re;
      mr[256 * 15] += R.muv.im;
    }
  }
  // the source geometry is read again here rather than held in registers
  // through the lattice sums (the empty asm hides the earlier load)
  const TetGeom *tgs = tg + S;
  asm volatile("" : "+v"(tgs));
  const TetGeom gs = *tgs;
  scatter_tt(M, gt, gs, t2f, T, S, alpha, gsrc, kappa, k0sq9, out, false);
  if (REV && sym) {
    Moments R;
    R.m0 = mk(mr[0], mr[256]);
    for (int d = 0; d < 3; ++d) {
      R.mu[d] = mk(mr[256 * (2 + 2 * d)], mr[256 * (3 + 2 * d)]);
      R.mv[d] = mk(mr[256 * (8 + 2 * d)], mr[256 * (9 + 2 * d)]);
    }
    R.muv = mk(mr[256 * 14], mr[256 * 15]);
    scatter_tt<true>(R, gs, gt, t2f, S, T, alpha, gsrc, kappa, k0sq9, outT, false);
  } else if (sym) {
    // (S, T) at kt = 0: test offsets and source offsets trade places
    Moments Ms;
    Ms.m0 = M.m0;
    Ms.muv = M.muv;
    for (int d = 0; d < 3; ++d) {
      Ms.mu[d] = M.mv[d];
      Ms.mv[d] = M.mu[d];
    }
    scatter_tt<true>(Ms, gs, gt, t2f, S, T, alpha, gsrc, kappa, k0sq9, outT, false);
  }
}

// ------------------------------------------------------------ pairs with faces
// M0 = II g_p over (test tet T, face F), 4 x 3 points: one face point against
// the tet's four points per lattice-sum call.
__device__ dz far_tet_face_c(const double *__restrict__ P, const QuadRules *__restrict__ qr, const TetGeom &gt,
                             const FaceGeom &f) {
  double fp[3][3];
  for (int j = 0; j < 3; ++j)
    for (int d = 0; d < 3; ++d) fp[j][d] = qr->tri3[j][0] * f.v[0][d] + qr->tri3[j][1] * f.v[1][d] + qr->tri3[j][2] * f.v[2][d];
  const double wf = f.area / 3.0;
  dz acc = mk(0, 0);
  double tp[4][3];
  for (int i = 0; i < 4; ++i)
    for (int d = 0; d < 3; ++d) {
      double s = 0;
      for (int k = 0; k < 4; ++k) s = fma(qr->tet4[i][k], gt.v[k][d], s);
      tp[i][d] = s;
    }
#pragma unroll 1
  for (int j = 0; j < 3; ++j) {
    double sep[4][3];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int d = 0; d < 3; ++d) sep[i][d] = tp[i][d] - fp[j][d];
    dz g[4];
    pgf_fixed_w<4>(P, sep, g);
    acc = acc + ((g[0] + g[1]) + (g[2] + g[3]));
  }
  return (0.25 * gt.vol * wf) * acc;
}

// M0 = II g_p over (test face F, source tet S), 3 x 4 points.
__device__ dz far_face_tet_c(const double *__restrict__ P, const QuadRules *__restrict__ qr, const FaceGeom &f,
                             const TetGeom &gs) {
  double sp[4][3];
  for (int j = 0; j < 4; ++j)
    for (int d = 0; d < 3; ++d) {
      double s = 0;
      for (int k = 0; k < 4; ++k) s = fma(qr->tet4[j][k], gs.v[k][d], s);
      sp[j][d] = s;
    }
  const double ws = 0.25 * gs.vol;
  dz acc = mk(0, 0);
#pragma unroll 1
  for (int i = 0; i < 3; ++i) {
    double r[3];
    for (int d = 0; d < 3; ++d) r[d] = qr->tri3[i][0] * f.v[0][d] + qr->tri3[i][1] * f.v[1][d] + qr->tri3[i][2] * f.v[2][d];
    double sep[4][3];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int d = 0; d < 3; ++d) sep[j][d] = r[d] - sp[j][d];
    dz g[4];
    pgf_fixed_w<4>(P, sep, g);
    acc = acc + ((g[0] + g[1]) + (g[2] + g[3]));
  }
  return (f.area / 3.0 * ws) * acc;
}

// M0 = II g_p over (test face F, source face G), 3 x 3 points.
__device__ dz far_face_face_c(const double *__restrict__ P, const QuadRules *__restrict__ qr, const FaceGeom &f,
                              const FaceGeom &g) {
  double gp[3][3];
  for (int j = 0; j < 3; ++j)
    for (int d = 0; d < 3; ++d) gp[j][d] = qr->tri3[j][0] * g.v[0][d] + qr->tri3[j][1] * g.v[1][d] + qr->tri3[j][2] * g.v[2][d];
  const double wg = g.area / 3.0;
  dz acc = mk(0, 0);
#pragma unroll 1
  for (int i = 0; i < 3; ++i) {
    double r[3];
    for (int d = 0; d < 3; ++d) r[d] = qr->tri3[i][0] * f.v[0][d] + qr->tri3[i][1] * f.v[1][d] + qr->tri3[i][2] * f.v[2][d];
    double sep[3][3];
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
      for (int d = 0; d < 3; ++d) sep[j][d] = r[d] - gp[j][d];
    dz v[3];
    pgf_fixed_w<3>(P, sep, v);
    acc = acc + (v[0] + v[1]) + v[2];
  }
  return (f.area / 3.0 * wg) * acc;
}

// far_tet_face_c and its value at the reversed separations (test face, source
// tet) from one lattice sum (oblique incidence).
__device__ void far_tet_face_rev_c(const double *__restrict__ P, const QuadRules *__restrict__ qr,
                                   const TetGeom &gt, const FaceGeom &f, dz &m0, dz &m0r) {
  double fp[3][3], tp[4][3];
  for (int j = 0; j < 3; ++j)
    for (int d = 0; d < 3; ++d) fp[j][d] = qr->tri3[j][0] * f.v[0][d] + qr->tri3[j][1] * f.v[1][d] + qr->tri3[j][2] * f.v[2][d];
  for (int i = 0; i < 4; ++i)
    for (int d = 0; d < 3; ++d) {
      double s = 0;
      for (int k = 0; k < 4; ++k) s = fma(qr->tet4[i][k], gt.v[k][d], s);
      tp[i][d] = s;
    }
  dz acc = mk(0, 0), accr = mk(0, 0);
#pragma unroll 1
  for (int j = 0; j < 3; ++j) {
    double sep[4][3];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int d = 0; d < 3; ++d) sep[i][d] = tp[i][d] - fp[j][d];
    dz g[4], gr[4];
    pgf_fixed_w<4, true>(P, sep, g, gr);
    acc = acc + ((g[0] + g[1]) + (g[2] + g[3]));
    accr = accr + ((gr[0] + gr[1]) + (gr[2] + gr[3]));
  }
  const double w = 0.25 * gt.vol * (f.area / 3.0);
  m0 = w * acc;
  m0r = w * accr;
}

// test tet (colour class list) x surface-charge face, far pairs, and with swap
// set the (half-SWG face, tet) entries into outT (see k_tet_face in k_fill.hip)
template <bool REV>
__device__ __forceinline__ void tet_face_c_body(const double *__restrict__ pack, int packlen, const QuadRules *__restrict__ qr,
                                                const TetGeom *__restrict__ tg, const TetFace *__restrict__ t2f,
                                                const int32_t *__restrict__ test_list, int ntest,
                                                const FaceGeom *__restrict__ fg, int nface,
                                                const dz *__restrict__ alpha, const dz *__restrict__ sigma,
                                                const dz *__restrict__ gsrc, const dz *__restrict__ kappa,
                                                ZOut out, ZOut outT, int swap, int bx_, int by_) {
  extern __shared__ double s_tab[];
  stage_table(pack, packlen, s_tab);

  const int ti = uniform(by_ * 4 + (threadIdx.x >> 6));
  const int fi = bx_ * 64 + (threadIdx.x & 63);
  if (ti >= ntest || fi >= nface) return;
  const int T = uniform(test_list[ti]);
  const TetGeom &gt = tg[T];
  const FaceGeom f = fg[fi];
  if (touch_mask(gt.canon, gt.off, 4, f.canon, f.off, 3)) return;
  dz m0, m0r;
  if (REV) {
    far_tet_face_rev_c(s_tab, qr, gt, f, m0, m0r);
  } else {
    m0 = far_tet_face_c(s_tab, qr, gt, f);
    m0r = m0;
  }
  const dz sm = sigma[fi] * m0;
  for (int k = 0; k < 4; ++k) zput(out, t2f[4 * T + k].unknown, f.unknown, mk(0, 0) - alpha[4 * T + k] * sm, false);
  if (swap && f.half) {
    const dz km = m0r * kappa[T];
    for (int l = 0; l < 4; ++l) zput(outT, t2f[4 * T + l].unknown, f.unknown, mk(0, 0) - gsrc[4 * T + l] * km, false);
  }
}

// half-SWG test face x source tet (colour class list), far pairs
__device__ __forceinline__ void face_tet_c_body(const double *__restrict__ pack, int packlen, const QuadRules *__restrict__ qr,
                                                const FaceGeom *__restrict__ fg, const int32_t *__restrict__ half_list,
                                                int nhalf, const TetGeom *__restrict__ tg,
                                                const TetFace *__restrict__ t2f, const int32_t *__restrict__ src_list,
                                                int nsrc, const dz *__restrict__ gsrc, const dz *__restrict__ kappa,
                                                ZOut out, int bx_, int by_) {
  extern __shared__ double s_tab[];
  stage_table(pack, packlen, s_tab);

  const int hi = uniform(by_ * 4 + (threadIdx.x >> 6));
  const int si = bx_ * 64 + (threadIdx.x & 63);
  if (hi >= nhalf || si >= nsrc) return;
  const FaceGeom &f = fg[uniform(half_list[hi])];
  const int S = src_list[si];
  const TetGeom gs = tg[S];
  if (touch_mask(f.canon, f.off, 3, gs.canon, gs.off, 4)) return;
  const dz m0 = far_face_tet_c(s_tab, qr, f, gs) * kappa[S];
  for (int l = 0; l < 4; ++l) zput(out, f.unknown, t2f[4 * S + l].unknown, mk(0, 0) - gsrc[4 * S + l] * m0, false);
}

// half-SWG test face x surface-charge face, far pairs
__device__ __forceinline__ void face_face_c_body(const double *__restrict__ pack, int packlen, const QuadRules *__restrict__ qr,
                                                 const FaceGeom *__restrict__ fg,
                                                 const int32_t *__restrict__ half_list, int nhalf, int nface,
                                                 const dz *__restrict__ sigma, ZOut out, int bx_, int by_) {
  extern __shared__ double s_tab[];
  stage_table(pack, packlen, s_tab);

  const int hi = uniform(by_ * 4 + (threadIdx.x >> 6));
  const int gi = bx_ * 64 + (threadIdx.x & 63);
  if (hi >= nhalf || gi >= nface) return;
  const FaceGeom &f = fg[uniform(half_list[hi])];
  const FaceGeom g = fg[gi];
  if (touch_mask(f.canon, f.off, 3, g.canon, g.off, 3)) return;
  zput(out, f.unknown, g.unknown, sigma[gi] * far_face_face_c(s_tab, qr, f, g), false);
}

// ------------------------------------------------------------ launches
// One segment per cell (a single context launches one): see FarSeg.
template <bool REV>
__device__ __forceinline__ void far_seg_c(const FarSeg &A, int bx, int by) {
  tt_far_c_body<REV>(A.pack, A.packlen, A.qr, A.tg, A.t2f, A.test_list, A.ntest, A.src_list, A.nsrc, A.alpha, A.gsrc,
                     A.kappa, A.k0sq9, A.out, A.outT, A.sym, bx, by);
}
template <bool REV>
__device__ __forceinline__ void tet_face_seg_c(const TetFaceSeg &A, int bx, int by) {
  tet_face_c_body<REV>(A.pack, A.packlen, A.qr, A.tg, A.t2f, A.test_list, A.ntest, A.fg, A.nface, A.alpha, A.sigma,
                       A.gsrc, A.kappa, A.out, A.outT, A.swap, bx, by);
}
__device__ __forceinline__ void face_tet_seg_c(const FaceTetSeg &A, int bx, int by) {
  face_tet_c_body(A.pack, A.packlen, A.qr, A.fg, A.half_list, A.nhalf, A.tg, A.t2f, A.src_list, A.nsrc, A.gsrc,
                  A.kappa, A.out, bx, by);
}
__device__ __forceinline__ void face_face_seg_c(const FaceFaceSeg &A, int bx, int by) {
  face_face_c_body(A.pack, A.packlen, A.qr, A.fg, A.half_list, A.nhalf, A.nface, A.sigma, A.out, bx, by);
}

// (kernel arguments for one cell, a table of segments for a batch)
#define VIE_FAR_C(NAME, SEG, BODY)                                                                    \
  __global__ __launch_bounds__(256, 2) void NAME(SEG A) { BODY(A, blockIdx.x, blockIdx.y); }          \
  __global__ __launch_bounds__(256, 2) void NAME##_seg(const SEG *__restrict__ segs, int nseg) {      \
    VIE_SEG_BEGIN(SEG)                                                                                \
    BODY(A, bx, by);                                                                                  \
  }
VIE_FAR_C(k_tt_far_c, FarSeg, far_seg_c<false>)
VIE_FAR_C(k_tt_far_rev_c, FarSeg, far_seg_c<true>)
VIE_FAR_C(k_tet_face_c, TetFaceSeg, tet_face_seg_c<false>)
VIE_FAR_C(k_tet_face_rev_c, TetFaceSeg, tet_face_seg_c<true>)
VIE_FAR_C(k_face_tet_c, FaceTetSeg, face_tet_seg_c)
VIE_FAR_C(k_face_face_c, FaceFaceSeg, face_face_seg_c)
#undef VIE_FAR_C

}  // namespace vie
