// Far element pairs of the mixed-precision operator (FP32 entries).
//
// Every contribution is added to its FP32 entry in FP64 and rounded, so a
// contribution that moves by a few 1e-16 moves isolated entries to the
// neighbouring FP32 value: 1e-7 of them, which leaves Z x within 3e-11 and the
// solution within 1e-9 in norm, but a single component of it 1e-7 off (N =
// 37,376).  A path that solves to 1e-12 should not move by that with the form
// of a series, so the arithmetic of these contributions is held fixed, to the
// bit: the terms come from one evaluation (PgfTerms::fixed), each as its
// Chebyshev series by Clenshaw's recurrence; images and orders are summed in
// the order of their grids, and the point pairs of an element pair one after
// the other.  k_fill.hip, whose entries are FP64, is free of this and takes
// whichever form is fastest; touching pairs are FP64 in both paths and come
// from there.
//
// Which lane forms which values is free.  Four lanes share a tet pair, which
// matters for small cells, where a launch is one lane's chain: far pairs of N =
// 416, symmetric, 10 launches, 0.60 ms, 3.8 with one lane per pair; N = 3,038 3.4
// against 5.5.  The series' coefficients come through the scalar cache into
// scalar registers (the table in LDS, the same lanes: 419 ms at N = 37,376), and
// the values of a pair wait in LDS, not in registers, for its moments (357; the
// reversed form spilled 284 B per lane).  Now 332 ms there (407 with one lane per
// pair, padded series and the table in LDS): 3,940 vector instructions per point
// pair and wave, 3,410 of them FP64 (an addition and an FMA per degree and term;
// 2,700 and 1,870 in k_fill.hip), issued at 82 % of the rate at 2.4 GHz.
#include "fill.h"

namespace vie {

// Packed table of these kernels (pack_pgf_fixed), read through the scalar cache:
// every address is the same in all lanes, and a coefficient that is in scalar
// registers takes no vector registers, no LDS reads and no moves.
typedef const double __attribute__((address_space(4))) *FixedTab;
__device__ __forceinline__ FixedTab fixed_tab(const double *p) { return (FixedTab)(uintptr_t)p; }
namespace pkf {
constexpr int A = 1, B = 2, IA = 3, IB = 4, E = 0, KX = 5, KY = 6, TPA = 7, TPB = 8, WS = 9, PHRE = 10, PHIM = 19,
              MMAX = 28, NMAX = kFixedNmax, ROWS = kFixedRows, RECORDS = kFixedRecords;
}
__device__ __forceinline__ int lo32(double v) { return ufirst(__double2loint(v)); }
__device__ __forceinline__ int hi32(double v) { return ufirst(__double2hiint(v)); }

// (scalar loads return in any order: those under way are waited for before the next are asked for)
__device__ __forceinline__ void scalar_wait() {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
  __builtin_amdgcn_sched_barrier(0);
}

// A Chebyshev series [K, c_K, c_{K-1}, c_{K-2} - c_K | c_{K-3} .. c_0] (K even, >= 4)
// in the table: its first eight values, and where the others are.
struct FixedSeries {
  double v[8];
  FixedTab q;
};
__device__ __forceinline__ FixedSeries fixed_series(FixedTab q) {
  FixedSeries s;
#pragma unroll
  for (int i = 0; i < 8; ++i) s.v[i] = q[i];
  s.q = q + 8;
  return s;
}

// The series at NC arguments t (t2 = 2 t) by Clenshaw's recurrence b_k = 2 t
// b_{k+1} + (c_k - b_{k+2}), f = t b_1 + (c_0 - b_2): each coefficient is read
// once for all of them, four at a time, the next four while the current ones are
// used.  The first two steps, whose b are zero or c_K, are formed without them.
template <int NC>
__device__ __forceinline__ void clenshaw(const FixedSeries &s, const double (&t)[NC], const double (&t2)[NC],
                                         double (&f)[NC]) {
  FixedTab q = s.q;
  double e0 = s.v[4], e1 = s.v[5], e2 = s.v[6], e3 = s.v[7];
  int r = lo32(s.v[0]) - 2;   // coefficients from e0 on
  double b1[NC], b2[NC];
#pragma unroll
  for (int i = 0; i < NC; ++i) b2[i] = fma(t2[i], s.v[1], s.v[2]);
#pragma unroll
  for (int i = 0; i < NC; ++i) b1[i] = fma(t2[i], b2[i], s.v[3]);
  const auto step = [&](double c, double (&n)[NC], const double (&o)[NC]) {   // n: b_{k+2}, then b_k
#pragma unroll
    for (int i = 0; i < NC; ++i) n[i] = fma(t2[i], o[i], c - n[i]);
  };
#pragma unroll 1
  for (; r > 4; r -= 4) {
    scalar_wait();
    const double n0 = q[0], n1 = q[1], n2 = q[2], n3 = q[3];
    q += 4;
    step(e0, b2, b1);
    step(e1, b1, b2);
    step(e2, b2, b1);
    step(e3, b1, b2);
    e0 = n0;
    e1 = n1;
    e2 = n2;
    e3 = n3;
  }
  if (r == 4) {
    step(e0, b2, b1);
    step(e1, b1, b2);
    e0 = e2;
    e1 = e3;
  }
  step(e0, b2, b1);
#pragma unroll
  for (int i = 0; i < NC; ++i) f[i] = fma(t[i], b2[i], e1 - b1[i]);
}

// g_p at W separations d[w] = r - r'_w of non-touching elements (one point
// against W), from the packed table P: images (m, n), then orders (p, q), each
// added in the order of its grid.
// REV: also g_p at -d[w] into rev[w] (see pgf_eval_w).
template <int W, bool REV = false>
__device__ __forceinline__ void pgf_fixed_w(FixedTab P, const double (&d)[W][3], dz (&out)[W], dz *rev = nullptr) {
  const double a = P[pkf::A], b = P[pkf::B], E = P[pkf::E];
  double dx[W], dy[W], dz2[W], sre[W], sim[W];
  int shift[W];   // the nearest image's phase
#pragma unroll
  for (int w = 0; w < W; ++w) {
    const double m0 = rint(d[w][0] * P[pkf::IA]), n0 = rint(d[w][1] * P[pkf::IB]);
    dx[w] = fma(-m0, a, d[w][0]);
    dy[w] = fma(-n0, b, d[w][1]);
    dz2[w] = d[w][2] * d[w][2];
    shift[w] = ((int)m0 + 1) * 3 + ((int)n0 + 1);
    sre[w] = 0.0;
    sim[w] = 0.0;
  }
  // the records, one after the other: the images in the order of (m, n)
  FixedTab q = P + pkf::RECORDS;
  const int mmax = lo32(P[pkf::MMAX]);
#pragma unroll 1
  for (int m = -mmax; m <= mmax; ++m) {
    const int nmax = lo32(P[pkf::NMAX + (m < 0 ? -m : m)]);
    double X[W];
#pragma unroll
    for (int w = 0; w < W; ++w) X[w] = fma((double)m, a, dx[w]);
#pragma unroll 1
    for (int n = -nmax; n <= nmax; ++n) {
      // [E xs, -(xa xs + 1), Re, Im phase], the F series
      scalar_wait();
      const double ts = q[0], t0 = q[1], cre = q[2], cim = q[3];
      const FixedSeries fs = fixed_series(q + 4);
      __builtin_amdgcn_sched_barrier(0);   // (asked for before the distances are formed)
      double t[W], t2[W], sc[W], f[W];
#pragma unroll
      for (int w = 0; w < W; ++w) {
        const double Y = fma((double)n, b, dy[w]);
        const double R2 = fma(X[w], X[w], fma(Y, Y, dz2[w]));
        sc[w] = rsqrt_pos(R2);
        t[w] = fma(R2 * sc[w], ts, t0);
        t2[w] = t[w] + t[w];
      }
      clenshaw<W>(fs, t, t2, f);
#pragma unroll
      for (int w = 0; w < W; ++w) {
        const double g = f[w] * sc[w];
        sre[w] = fma(cre, g, sre[w]);
        sim[w] = fma(cim, g, sim[w]);
      }
      q += hi32(fs.v[0]);
    }
  }

  // then the orders in the order of (p, q): the W separations share every
  // series; the Floquet phases e^{-j k_tpq . Delta_t} of each separation by
  // recurrence in p and q
  double tw[W], tw2[W], kre[W], kim[W], cre_[W], cim_[W];
  dz erow[W], bx[W], by[W];   // erow: phase of (p, q = -4); steps in p and in q
  const bool kt0 = P[pkf::KX] == 0.0 && P[pkf::KY] == 0.0;   // normal incidence: e^{-j kt.Delta} = 1
#pragma unroll
  for (int w = 0; w < W; ++w) {
    tw[w] = fma(dz2[w] * E * E, P[pkf::WS], -1.0);
    tw2[w] = tw[w] + tw[w];
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
#pragma unroll 1
  for (int p = 0; p < kPgfSide; ++p) {
    // slots with an order, and with an imaginary part; none past the last of them is visited
    int any = lo32(P[pkf::ROWS + p]), cplx = hi32(P[pkf::ROWS + p]);
    dz e[W];
#pragma unroll
    for (int w = 0; w < W; ++w) e[w] = erow[w];
#pragma unroll 1
    for (; any != 0; any >>= 1, cplx >>= 1) {
      scalar_wait();
      const FixedSeries re = fixed_series(q);   // (of a later slot if this one has no order)
      __builtin_amdgcn_sched_barrier(0);
      if (any & 1) {
        double kr[W];
        clenshaw<W>(re, tw, tw2, kr);
        q += hi32(re.v[0]);
        if (cplx & 1) {
          double ki[W];
          const FixedSeries im = fixed_series(q);
          clenshaw<W>(im, tw, tw2, ki);
          q += hi32(im.v[0]);
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
    const dz ph = mk(P[pkf::PHRE + shift[w]], P[pkf::PHIM + shift[w]]);
    out[w] = ph * mk(sre[w] + kre[w], sim[w] + kim[w]);
    if (REV) rev[w] = conjz(out[w]) + conjz(ph) * mk(-2.0 * cim_[w], 2.0 * cre_[w]);
  }
}

// Z[m][n] += v, formed in FP64 and rounded.
__device__ __forceinline__ void zput_c(const ZOut &o, int64_t m, int64_t n, dz v) {
  fz *p = o.Zs + m * o.ld + n;
  const fz z = *p;
  *p = fz{(float)((double)z.re + v.re), (float)((double)z.im + v.im)};
}

// Row k of the contributions of tet pair (T, S) to Z (TRANS: entry (m, n)
// goes to (n, m) of the output).
template <bool TRANS>
__device__ __forceinline__ void scatter_tt_row_c(const Moments &M, const TetGeom &gt, const TetGeom &gs,
                                                 const TetFace *__restrict__ t2f, int T, int S, int k,
                                                 const dz *__restrict__ alpha, const dz *__restrict__ gsrc,
                                                 const dz *__restrict__ kappa, double k0sq9, const ZOut &out) {
  const dz ks = kappa[S];
  double pk[3];
  for (int d = 0; d < 3; ++d) pk[d] = gt.v[k][d] - gt.c[d];
  // muv - p~.mv
  dz base = M.muv;
  for (int d = 0; d < 3; ++d) base = base - pk[d] * M.mv[d];
  const dz ak = alpha[4 * T + k];
  const int64_t row = t2f[4 * T + k].unknown;
#pragma unroll 2
  for (int l = 0; l < 4; ++l) {
    double qv[3];
    for (int d = 0; d < 3; ++d) qv[d] = gs.v[l][d] - gs.c[d];
    const dz bl = gsrc[4 * S + l] * ks;
    const int64_t col = t2f[4 * S + l].unknown;
    dz I = base;
    for (int d = 0; d < 3; ++d) I = I - qv[d] * M.mu[d];
    I = I + dot3(pk, qv) * M.m0;
    const dz v = M.m0 - k0sq9 * I;
    if (TRANS) zput_c(out, col, row, (ak * bl) * v);
    else zput_c(out, row, col, (ak * bl) * v);
  }
}

// Far tet pairs: 4 x 4 product rule, four lanes per pair, lane i the test point
// i against the four source points.  The sixteen values meet in LDS (the pairs of
// a wave 33 values apart: no bank conflicts), and every lane of the four takes
// them in the order of the points into all moments (its own copy) and writes
// the entries of one test face.  A wave takes 16 sources, a block 64
// and one test tet.  sym > 0 writes the swapped pair's block (S, T)
// too, from the pair's own moments at normal incidence, else (REV) from those of
// the reversed separations.
template <bool REV>
__device__ __forceinline__ void tt_far_c_body(FixedTab P, const QuadRules *__restrict__ qr, const TetGeom *__restrict__ tg,
                                              const TetFace *__restrict__ t2f, const int32_t *__restrict__ test_list,
                                              const int32_t *__restrict__ src_list, int nsrc,
                                              const dz *__restrict__ alpha, const dz *__restrict__ gsrc,
                                              const dz *__restrict__ kappa, double k0sq9, const ZOut &out,
                                              const ZOut &outT, int sym, int bx_, int by_) {
  // one list against itself: pairs with the source position above the test position
  const int ti = by_;
  if (sym == 2 && bx_ * 64 + 63 <= ti) return;
  const int k = threadIdx.x & 3;
  const int si = bx_ * 64 + (threadIdx.x >> 2);
  const int S = src_list[min(si, nsrc - 1)];
  const TetGeom *gs = tg + S;
  const int T = uniform(test_list[ti]);
  const TetGeom &gt = tg[T];
  bool act = si < nsrc && (sym != 2 || si > ti);
  {
    // touching pairs (a shared vertex under any image): k_tt_near; lane k looks at the test vertex k
    const int32_t ct = gt.canon[k];
    const bool hit = ct == gs->canon[0] || ct == gs->canon[1] || ct == gs->canon[2] || ct == gs->canon[3];
    act = act && ((__ballot(hit) >> (threadIdx.x & 60)) & 15) == 0;
  }
  if (__ballot(act) == 0) return;
  __shared__ dz s_g[64 * (REV ? 33 : 17)];
  dz *mine = s_g + (threadIdx.x >> 2) * (REV ? 33 : 17);
  {
    dz g[4], gr[4];
    double sep[4][3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      double s = 0;
      for (int q = 0; q < 4; ++q) s = fma(qr->tet4[k][q], gt.v[q][d], s);
      const double u = s - gt.c[d], dc = gt.c[d] - gs->c[d];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        double r = 0;
        for (int q = 0; q < 4; ++q) r = fma(qr->tet4[j][q], gs->v[q][d], r);
        sep[j][d] = dc + u - (r - gs->c[d]);
      }
    }
    pgf_fixed_w<4, REV>(P, sep, g, gr);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      mine[4 * k + j] = g[j];
      if (REV) mine[16 + 4 * k + j] = gr[j];
    }
  }
  __builtin_amdgcn_wave_barrier();   // (a wave reads what it wrote)
  const double wt = 0.25 * gt.vol;
  // source points relative to the source centroid.  The source geometry is read
  // again for each use rather than held in registers through the lattice sums
  // and the stores (the empty asm hides the earlier loads).
  const auto sources = [&](double (&up)[4][3]) {
    asm volatile("" : "+v"(gs));
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        double s = 0;
        for (int q = 0; q < 4; ++q) s = fma(qr->tet4[j][q], gs->v[q][d], s);
        up[j][d] = s - gs->c[d];
      }
  };
  const auto test_point = [&](int i, double (&u)[3]) {   // relative to the test centroid
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      double s = 0;
      for (int q = 0; q < 4; ++q) s = fma(qr->tet4[i][q], gt.v[q][d], s);
      u[d] = s - gt.c[d];
    }
  };
  {
    double up[4][3];
    sources(up);
    const double wq = 0.25 * gs->vol;
    Moments M;
    moments_zero(M);
#pragma unroll 1
    for (int i = 0; i < 4; ++i) {
      double u[3];
      test_point(i, u);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const dz gw = (wt * wq) * mine[4 * i + j];
        M.m0 = M.m0 + gw;
        for (int d = 0; d < 3; ++d) {
          axpy(M.mu[d], u[d], gw);
          axpy(M.mv[d], up[j][d], gw);
        }
        axpy(M.muv, dot3(u, up[j]), gw);
      }
    }
    if (act) {
      scatter_tt_row_c<false>(M, gt, *gs, t2f, T, S, k, alpha, gsrc, kappa, k0sq9, out);
      if (!REV && sym) {
        // (S, T) at kt = 0: test offsets and source offsets trade places
        Moments Ms;
        Ms.m0 = M.m0;
        Ms.muv = M.muv;
        for (int d = 0; d < 3; ++d) {
          Ms.mu[d] = M.mv[d];
          Ms.mv[d] = M.mu[d];
        }
        scatter_tt_row_c<true>(Ms, *gs, gt, t2f, S, T, k, alpha, gsrc, kappa, k0sq9, outT);
      }
    }
  }
  if (REV) {
    // swapped pair (S, T): its test offsets are up_j, its source offsets u;
    // the moments of each test point are summed by themselves first
    double up[4][3];
    sources(up);
    const double wq = 0.25 * gs->vol;
    Moments Mr;
    moments_zero(Mr);
#pragma unroll 1
    for (int i = 0; i < 4; ++i) {
      double u[3];
      test_point(i, u);
      Moments R;
      moments_zero(R);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const dz grw = (wt * wq) * mine[16 + 4 * i + j];
        R.m0 = R.m0 + grw;
        for (int d = 0; d < 3; ++d) {
          axpy(R.mu[d], up[j][d], grw);
          axpy(R.mv[d], u[d], grw);
        }
        axpy(R.muv, dot3(u, up[j]), grw);
      }
      Mr.m0 = Mr.m0 + R.m0;
      for (int d = 0; d < 3; ++d) {
        Mr.mu[d] = Mr.mu[d] + R.mu[d];
        Mr.mv[d] = Mr.mv[d] + R.mv[d];
      }
      Mr.muv = Mr.muv + R.muv;
    }
    if (act) scatter_tt_row_c<true>(Mr, *gs, gt, t2f, S, T, k, alpha, gsrc, kappa, k0sq9, outT);
  }
}

// ------------------------------------------------------------ pairs with faces
// M0 = II g_p over (test tet T, face F), 4 x 3 points: one face point against
// the tet's four points per lattice-sum call.
__device__ dz far_tet_face_c(FixedTab P, const QuadRules *__restrict__ qr, const TetGeom &gt,
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
__device__ dz far_face_tet_c(FixedTab P, const QuadRules *__restrict__ qr, const FaceGeom &f,
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
__device__ dz far_face_face_c(FixedTab P, const QuadRules *__restrict__ qr, const FaceGeom &f,
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
__device__ void far_tet_face_rev_c(FixedTab P, const QuadRules *__restrict__ qr,
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
__device__ __forceinline__ void tet_face_c_body(FixedTab P, const QuadRules *__restrict__ qr,
                                                const TetGeom *__restrict__ tg, const TetFace *__restrict__ t2f,
                                                const int32_t *__restrict__ test_list, int ntest,
                                                const FaceGeom *__restrict__ fg, int nface,
                                                const dz *__restrict__ alpha, const dz *__restrict__ sigma,
                                                const dz *__restrict__ gsrc, const dz *__restrict__ kappa,
                                                ZOut out, ZOut outT, int swap, int bx_, int by_) {
  const int ti = uniform(by_ * 4 + (threadIdx.x >> 6));
  const int fi = bx_ * 64 + (threadIdx.x & 63);
  if (ti >= ntest || fi >= nface) return;
  const int T = uniform(test_list[ti]);
  const TetGeom &gt = tg[T];
  const FaceGeom f = fg[fi];
  if (touch_mask(gt.canon, gt.off, 4, f.canon, f.off, 3)) return;
  dz m0, m0r;
  if (REV) {
    far_tet_face_rev_c(P, qr, gt, f, m0, m0r);
  } else {
    m0 = far_tet_face_c(P, qr, gt, f);
    m0r = m0;
  }
  const dz sm = sigma[fi] * m0;
  for (int k = 0; k < 4; ++k) zput_c(out, t2f[4 * T + k].unknown, f.unknown, mk(0, 0) - alpha[4 * T + k] * sm);
  if (swap && f.half) {
    const dz km = m0r * kappa[T];
    for (int l = 0; l < 4; ++l) zput_c(outT, t2f[4 * T + l].unknown, f.unknown, mk(0, 0) - gsrc[4 * T + l] * km);
  }
}

// half-SWG test face x source tet (colour class list), far pairs
__device__ __forceinline__ void face_tet_c_body(FixedTab P, const QuadRules *__restrict__ qr,
                                                const FaceGeom *__restrict__ fg, const int32_t *__restrict__ half_list,
                                                int nhalf, const TetGeom *__restrict__ tg,
                                                const TetFace *__restrict__ t2f, const int32_t *__restrict__ src_list,
                                                int nsrc, const dz *__restrict__ gsrc, const dz *__restrict__ kappa,
                                                ZOut out, int bx_, int by_) {
  const int hi = uniform(by_ * 4 + (threadIdx.x >> 6));
  const int si = bx_ * 64 + (threadIdx.x & 63);
  if (hi >= nhalf || si >= nsrc) return;
  const FaceGeom &f = fg[uniform(half_list[hi])];
  const int S = src_list[si];
  const TetGeom gs = tg[S];
  if (touch_mask(f.canon, f.off, 3, gs.canon, gs.off, 4)) return;
  const dz m0 = far_face_tet_c(P, qr, f, gs) * kappa[S];
  for (int l = 0; l < 4; ++l) zput_c(out, f.unknown, t2f[4 * S + l].unknown, mk(0, 0) - gsrc[4 * S + l] * m0);
}

// half-SWG test face x surface-charge face, far pairs
__device__ __forceinline__ void face_face_c_body(FixedTab P, const QuadRules *__restrict__ qr,
                                                 const FaceGeom *__restrict__ fg,
                                                 const int32_t *__restrict__ half_list, int nhalf, int nface,
                                                 const dz *__restrict__ sigma, ZOut out, int bx_, int by_) {
  const int hi = uniform(by_ * 4 + (threadIdx.x >> 6));
  const int gi = bx_ * 64 + (threadIdx.x & 63);
  if (hi >= nhalf || gi >= nface) return;
  const FaceGeom &f = fg[uniform(half_list[hi])];
  const FaceGeom g = fg[gi];
  if (touch_mask(f.canon, f.off, 3, g.canon, g.off, 3)) return;
  zput_c(out, f.unknown, g.unknown, sigma[gi] * far_face_face_c(P, qr, f, g));
}

// ------------------------------------------------------------ launches
// One segment per cell (a single context launches one): see FarSeg.
template <bool REV>
__device__ __forceinline__ void far_seg_c(const FarSeg &A, int bx, int by) {
  tt_far_c_body<REV>(fixed_tab(A.pack), A.qr, A.tg, A.t2f, A.test_list, A.src_list, A.nsrc, A.alpha, A.gsrc,
                     A.kappa, A.k0sq9, A.out, A.outT, A.sym, bx, by);
}
template <bool REV>
__device__ __forceinline__ void tet_face_seg_c(const TetFaceSeg &A, int bx, int by) {
  tet_face_c_body<REV>(fixed_tab(A.pack), A.qr, A.tg, A.t2f, A.test_list, A.ntest, A.fg, A.nface, A.alpha, A.sigma,
                       A.gsrc, A.kappa, A.out, A.outT, A.swap, bx, by);
}
__device__ __forceinline__ void face_tet_seg_c(const FaceTetSeg &A, int bx, int by) {
  face_tet_c_body(fixed_tab(A.pack), A.qr, A.fg, A.half_list, A.nhalf, A.tg, A.t2f, A.src_list, A.nsrc, A.gsrc,
                  A.kappa, A.out, bx, by);
}
__device__ __forceinline__ void face_face_seg_c(const FaceFaceSeg &A, int bx, int by) {
  face_face_c_body(fixed_tab(A.pack), A.qr, A.fg, A.half_list, A.nhalf, A.nface, A.sigma, A.out, bx, by);
}

// (kernel arguments for one cell, a table of segments for a batch)
#define VIE_FAR_C(NAME, SEG, BODY, WAVES)                                                                  \
  __global__ __launch_bounds__(256, WAVES) void NAME(SEG A) { BODY(A, blockIdx.x, blockIdx.y); }          \
  __global__ __launch_bounds__(256, WAVES) void NAME##_seg(const SEG *__restrict__ segs, int nseg) {      \
    VIE_SEG_BEGIN(SEG)                                                                                    \
    BODY(A, bx, by);                                                                                      \
  }
VIE_FAR_C(k_tt_far_c, FarSeg, far_seg_c<false>, 3)
VIE_FAR_C(k_tt_far_rev_c, FarSeg, far_seg_c<true>, 3)
VIE_FAR_C(k_tet_face_c, TetFaceSeg, tet_face_seg_c<false>, 3)
VIE_FAR_C(k_tet_face_rev_c, TetFaceSeg, tet_face_seg_c<true>, 2)
VIE_FAR_C(k_face_tet_c, FaceTetSeg, face_tet_seg_c, 3)
VIE_FAR_C(k_face_face_c, FaceFaceSeg, face_face_seg_c, 3)
#undef VIE_FAR_C

}  // namespace vie
