// Impedance-matrix fill of the periodic SWG VIE (Sec. 2.1, Eq. 2 with the
// periodic Green's function of Sec. 2.2, Eqs. 3-4), right-hand side, and a
// diagnostic evaluation of g_p.
//
// Galerkin terms for test tet T (local face k -> unknown m) and source tet S
// (local face l -> unknown n), u = r - c_T, u' = r' - c_S, p~ = v_k - c_T,
// q~ = v'_l - c_S:
//   Z_mn += alpha_Tk * beta_Sl * [ II g_p - (k0^2/9) II (u - p~).(u' - q~) g_p ]
//   alpha_Tk = chi s a_m / V_T,   beta_Sl = psi s a_n kappa_S / V_S,
// with the Bloch test/source phases chi = e^{+j kt.rho}, psi = e^{-j kt.rho} of
// a wall-shifted half.  Surface charges (sigma_n on interface/boundary faces)
// and the boundary term of half-SWG test faces add scalar-potential pairs of
// tetrahedra and faces.  The mass term <f_m, f_n/eps> is added with the
// self pair.
//
// Scatter: every launch covers a pair of tetrahedron colour classes (no two
// tetrahedra of a class share a face), so no two lanes of one launch touch
// the same Z entry; the read-modify-write needs no atomics and the result is
// deterministic.
#include <hip/hip_runtime.h>

#include "fill.h"

namespace vie {

// ------------------------------------------------------------ per-fill coefficients
__global__ void k_prep(int64_t nt, const TetFace *__restrict__ t2f, const TetGeom *__restrict__ tg,
                       const double *__restrict__ area, const dz *__restrict__ eps_int, double kx, double ky,
                       double a, double b, dz *__restrict__ alpha, dz *__restrict__ gsrc, dz *__restrict__ kappa,
                       dz *__restrict__ inv_eps) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= nt) return;
  const dz e = eps_int[t];
  const double den = e.re * e.re + e.im * e.im;
  const dz ie = mk(e.re / den, -e.im / den);
  inv_eps[t] = ie;
  kappa[t] = mk(1.0 - ie.re, -ie.im);
  const double V = tg[t].vol;
  for (int k = 0; k < 4; ++k) {
    const TetFace f = t2f[4 * t + k];
    double s, c;
    sincos(kx * f.sx * a + ky * f.sy * b, &s, &c);
    const double w = f.sign * area[f.unknown] / V;
    alpha[4 * t + k] = mk(w * c, w * s);   // e^{+j kt.rho} s a / V
    gsrc[4 * t + k] = mk(w * c, -w * s);   // e^{-j kt.rho} s a / V
  }
}

// sigma_n = kappa(T+) - kappa(T-) for each surface-charge face slot
__global__ void k_sigma(int nc, const int32_t *__restrict__ ctp, const int32_t *__restrict__ ctm,
                        const dz *__restrict__ kappa, dz *__restrict__ sigma) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nc) return;
  dz s = kappa[ctp[i]];
  if (ctm[i] >= 0) s = s - kappa[ctm[i]];
  sigma[i] = s;
}

__global__ void k_zero(dz *__restrict__ p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = mk(0.0, 0.0);
}

// ------------------------------------------------------------ tet-pair moments
// Lane sums by DPP moves: over a quad (quad swaps), and of lanes l and 7 - l
// of eight (half-row mirror).
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
  return v + __longlong_as_double((long long)dpp64<CTRL>((unsigned long long)__double_as_longlong(v)));
}
template <int CTRL>
__device__ __forceinline__ dz dpp_add(dz v) { return mk(dpp_add<CTRL>(v.re), dpp_add<CTRL>(v.im)); }
__device__ __forceinline__ dz quad_sum(dz v) { return dpp_add<0x4e>(dpp_add<0xb1>(v)); }
__device__ __forceinline__ dz mirror8_sum(dz v) { return dpp_add<0x141>(v); }
// over the wave, in every lane
__device__ __forceinline__ dz wave_sum64(dz v) {
  v = dpp_add<0x140>(mirror8_sum(quad_sum(v)));
  v = mk(v.re + __shfl_xor(v.re, 16), v.im + __shfl_xor(v.im, 16));
  return mk(v.re + __shfl_xor(v.re, 32), v.im + __shfl_xor(v.im, 32));
}

// Z_kl contributions of tet pair (T, S) from its moments: entries l0 .. l0 +
// nl - 1 of the test face k, entry (m, n) at (n, m) with trans.
__device__ __forceinline__ void scatter_tt_row(const Moments &M, const TetGeom &gt, const TetGeom &gs,
                                               const TetFace *__restrict__ t2f, int T, int S, int k, int l0, int nl,
                                               const dz *__restrict__ alpha, const dz *__restrict__ gsrc,
                                               const dz *__restrict__ kappa, double k0sq9, const ZOut &out, bool trans,
                                               bool near) {
  double pk[3];
  for (int d = 0; d < 3; ++d) pk[d] = gt.v[k][d] - gt.c[d];
  dz base = M.muv;   // muv - p~.mv
  for (int d = 0; d < 3; ++d) base = base - pk[d] * M.mv[d];
  const dz ak = alpha[4 * T + k] * kappa[S];
  const int64_t row = t2f[4 * T + k].unknown;
#pragma unroll 2
  for (int l = l0; l < l0 + nl; ++l) {
    double qv[3];
    for (int d = 0; d < 3; ++d) qv[d] = gs.v[l][d] - gs.c[d];
    dz I = base;
    for (int d = 0; d < 3; ++d) I = I - qv[d] * M.mu[d];
    I = I + dot3(pk, qv) * M.m0;
    const dz v = (ak * gsrc[4 * S + l]) * (M.m0 - k0sq9 * I);
    const int64_t col = t2f[4 * S + l].unknown;
    zput(out, trans ? col : row, trans ? row : col, v, near);
  }
}

// Far tet pairs: 4 x 4 product rule.  A wave takes one test tet at a time
// (tper of them in turn) against 8 source tets, eight lanes per pair: a lane
// takes one test point and two source points (lanes l and 7 - l the same test
// point).  The test point is fixed per lane, so the moments follow from sum g
// and sum g r' over the source points after the lattice sums, and none are
// held through them; after the sums each lane of a quad writes the entries of
// one test face.  Bound by the issue of FP64 instructions: at three waves a
// SIMD takes one every five cycles at best, 5,500 per wave (128 point pairs)
// run at 72 % of that.  N = 37,376, symmetric, oblique: 344 ms per fill, 442 ms
// with one lane per pair, the Clenshaw form of every series and one image at a
// time (pgf_eval_w); N = 18,590, ordered pairs: 145 ms, 196 before.  On small
// cells a launch's chain counts, an eighth of one lane per pair: N = 416, 16
// launches, 0.5 ms, 6.2 before.  (FP64 entries only: mixed precision takes
// k_far_c.hip.)
// sym > 0 writes the swapped pair's block (S, T) too (see the declaration):
// the second quad of the eight forms and writes it beside the first.  At
// normal incidence the lattice sum is even in the separation (the phases
// e^{-j kt.rho} are all 1), so the pair's moments also give those of the
// swapped pair.  At oblique incidence (REV) g_p at the reversed separations
// follows from g_p at the separations plus the propagating orders' term (see
// pgf_eval_w), and the swapped pair's moments are formed from it.
template <bool REV>
__device__ __forceinline__ void tt_far_body(const double *__restrict__ pack, int packlen,
                                            const QuadRules *__restrict__ qr, const TetGeom *__restrict__ tg,
                                            const TetFace *__restrict__ t2f, const int32_t *__restrict__ test_list,
                                            int ntest, const int32_t *__restrict__ src_list, int nsrc,
                                            const dz *__restrict__ alpha, const dz *__restrict__ gsrc,
                                            const dz *__restrict__ kappa, double k0sq9, const ZOut &out,
                                            const ZOut &outT, int sym, int tper, int bx_, int by_) {
  extern __shared__ double s_tab[];
  // one list against itself: a block whose source positions all lie at or
  // below its test positions has nothing to do (the whole block returns)
  if (sym == 2 && bx_ * 8 + 7 <= by_ * 4 * tper) return;
  stage_table(pack, packlen, s_tab);
  const int lane = threadIdx.x & 63, k = lane & 3;
  const bool second = (lane & 4) != 0;
  const int i = second ? 3 - k : k, j0 = second ? 2 : 0;   // test point, first source point
  const int si = bx_ * 8 + (lane >> 3);
  const int S = src_list[min(si, nsrc - 1)];
  double rs[2][3];   // the lane's source points
  int32_t canon[4];
  {
    const TetGeom gs = tg[S];
#pragma unroll
    for (int j = 0; j < 4; ++j) canon[j] = gs.canon[j];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        double s = 0;
        for (int q = 0; q < 4; ++q) s = fma(qr->tet4[j0 + j][q], gs.v[q][d], s);
        rs[j][d] = s;
      }
  }
#pragma unroll 1
  for (int tt = 0; tt < tper; ++tt) {
    const int ti = uniform((by_ * 4 + (threadIdx.x >> 6)) * tper + tt);
    if (ti >= ntest) return;
    const int T = uniform(test_list[ti]);
    const TetGeom &gt = tg[T];
    bool act = si < nsrc && (sym != 2 || si > ti);
    {
      // touching pairs (a shared vertex under any image): k_tt_near; lane k looks at the test vertex k
      const int32_t ct = gt.canon[k];
      const bool hit = ct == canon[0] || ct == canon[1] || ct == canon[2] || ct == canon[3];
      act = act && ((__ballot(hit) >> (lane & ~3)) & 15) == 0;
    }
    if (__ballot(act) == 0) continue;
    dz g[2], gr[2];
    {
      double sep[2][3];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        double s = 0;
        for (int q = 0; q < 4; ++q) s = fma(qr->tet4[i][q], gt.v[q][d], s);
        sep[0][d] = s - rs[0][d];
        sep[1][d] = s - rs[1][d];
      }
      pgf_eval_w<false, 2, REV>(s_tab, sep, 0, g, gr);
    }
    // the source geometry is read again here rather than held in registers
    // through the lattice sums (the empty asm hides the earlier load)
    const TetGeom *gs = tg + S;
    asm volatile("" : "+v"(gs));
    double u[3], v[2][3];   // test and source points relative to the centroids
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      double s = 0;
      for (int q = 0; q < 4; ++q) s = fma(qr->tet4[i][q], gt.v[q][d], s);
      u[d] = s - gt.c[d];
      v[0][d] = rs[0][d] - gs->c[d];
      v[1][d] = rs[1][d] - gs->c[d];
    }
    // sums over the four source points (of this lane and its mirror)
    dz G = mirror8_sum(g[0] + g[1]), G1[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) G1[d] = mirror8_sum(v[0][d] * g[0] + v[1][d] * g[1]);
    if (REV) {
      const dz H = mirror8_sum(gr[0] + gr[1]);
      G = second ? H : G;
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const dz H1 = mirror8_sum(v[0][d] * gr[0] + v[1][d] * gr[1]);
        G1[d] = second ? H1 : G1[d];
      }
    }
    // sums over the test points; (S, T): test and source offsets trade places
    const bool swap = sym && second;
    const double w = (0.25 * gt.vol) * (0.25 * gs->vol);
    Moments M;
    M.m0 = w * quad_sum(G);
    M.muv = mk(0, 0);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const dz a = w * quad_sum(u[d] * G), b = w * quad_sum(G1[d]);
      M.mu[d] = swap ? b : a;
      M.mv[d] = swap ? a : b;
      axpy(M.muv, u[d], G1[d]);
    }
    M.muv = w * quad_sum(M.muv);
    if (!act) continue;
    const TetGeom *ga = swap ? gs : &gt, *gb = swap ? &gt : gs;
    ZOut o = out;   // (out and outT differ in the dense part alone)
    o.Z = swap ? outT.Z : out.Z;
    o.Zs = swap ? outT.Zs : out.Zs;
    scatter_tt_row(M, *ga, *gb, t2f, swap ? S : T, swap ? T : S, k, sym ? 0 : j0, sym ? 4 : 2, alpha, gsrc, kappa, k0sq9,
                   o, swap, false);
  }
}

constexpr int kFarWaves = 3;   // waves per SIMD of the far kernels (two: 8 % slower; four spill, the same)
__global__ __launch_bounds__(256, kFarWaves) void k_tt_far(const double *__restrict__ pack, int packlen, const QuadRules *__restrict__ qr,
                                                const TetGeom *__restrict__ tg, const TetFace *__restrict__ t2f,
                                                const int32_t *__restrict__ test_list, int ntest,
                                                const int32_t *__restrict__ src_list, int nsrc,
                                                const dz *__restrict__ alpha, const dz *__restrict__ gsrc,
                                                const dz *__restrict__ kappa, double k0sq9, ZOut out, ZOut outT,
                                                int sym, int tper) {
  tt_far_body<false>(pack, packlen, qr, tg, t2f, test_list, ntest, src_list, nsrc, alpha, gsrc, kappa, k0sq9, out,
                     outT, sym, tper, blockIdx.x, blockIdx.y);
}

__global__ __launch_bounds__(256, kFarWaves) void k_tt_far_rev(const double *__restrict__ pack, int packlen, const QuadRules *__restrict__ qr,
                                                const TetGeom *__restrict__ tg, const TetFace *__restrict__ t2f,
                                                const int32_t *__restrict__ test_list, int ntest,
                                                const int32_t *__restrict__ src_list, int nsrc,
                                                const dz *__restrict__ alpha, const dz *__restrict__ gsrc,
                                                const dz *__restrict__ kappa, double k0sq9, ZOut out, ZOut outT,
                                                int sym, int tper) {
  tt_far_body<true>(pack, packlen, qr, tg, t2f, test_list, ntest, src_list, nsrc, alpha, gsrc, kappa, k0sq9, out,
                     outT, sym, tper, blockIdx.x, blockIdx.y);
}

// Z[i][j] += Zt[j][i]: 32 x 32 tiles through shared memory, both sides read
// and written along rows.  In FP32 the sum is formed in FP64 and rounded once.
template <typename C>
__device__ __forceinline__ void transpose_add_body(C *__restrict__ Z, const C *__restrict__ Zt, int64_t N, int64_t ld) {
  __shared__ C tile[32][33];
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 256 threads: 32 x 8
  const int64_t i0 = (int64_t)blockIdx.y * 32, j0 = (int64_t)blockIdx.x * 32;
  // tile of Zt rows j0.., columns i0..
  for (int r = ty; r < 32; r += 8) {
    const int64_t j = j0 + r, i = i0 + tx;
    if (j < N && i < N) tile[r][tx] = Zt[j * ld + i];
  }
  __syncthreads();
  for (int r = ty; r < 32; r += 8) {
    const int64_t i = i0 + r, j = j0 + tx;
    if (i < N && j < N) {
      const C a = Z[i * ld + j], b = tile[tx][r];
      Z[i * ld + j] = cx<C>::make((double)a.re + (double)b.re, (double)a.im + (double)b.im);
    }
  }
}
__global__ __launch_bounds__(256) void k_transpose_add_z(dz *Z, const dz *Zt, int64_t N, int64_t ld) {
  transpose_add_body(Z, Zt, N, ld);
}
__global__ __launch_bounds__(256) void k_transpose_add_c(fz *Z, const fz *Zt, int64_t N, int64_t ld) {
  transpose_add_body(Z, Zt, N, ld);
}

// Touching tet pairs: 14-point outer rule on T; per touching image the closed
// form int_S 1/R and int_S (r'-r)/R; 4-point inner rule for the remainder.
// The self pair also adds the mass term <f_m, f_n / eps_r>.  One wave per
// pair: lane 4 q + f takes the outer point q < 14 with the face f of S in the
// closed forms and the inner point f in the remainder (all of it adds up), the
// moments are summed over the wave, and lane 4 k + l writes entry (k, l).  A
// launch covers one colour pair, so on small cells its length is one lane's
// chain, and on large ones the waves in flight count, three per SIMD: N = 37,376,
// 13 ms per fill, 35 ms with 16 lanes per pair (the four faces and inner
// points in turn, 255 registers); N = 416, 0.5 ms, 1.7 before.
__device__ __forceinline__ void k_tt_near_body(const double *__restrict__ pack, int packlen, const QuadRules *__restrict__ qr,
                                                 const TetGeom *__restrict__ tg, const TetFace *__restrict__ t2f,
                                                 const int32_t *__restrict__ lt, const int32_t *__restrict__ ls,
                                                 const int32_t *__restrict__ lmask, int npairs,
                                                 const dz *__restrict__ alpha, const dz *__restrict__ gsrc,
                                                 const dz *__restrict__ kappa, const dz *__restrict__ inv_eps,
                                                 double k0sq9, ZOut out, int bx_, int by_) {
  extern __shared__ double s_tab[];
  stage_table(pack, packlen, s_tab);
  const double *__restrict__ P = s_tab;

  const int lane = threadIdx.x & 63, q = lane >> 2, f = lane & 3;
  const int pair = uniform(bx_ * 4 + (threadIdx.x >> 6));
  if (pair >= npairs) return;
  const int T = uniform(lt[pair]), S = uniform(ls[pair]), mask = uniform(lmask[pair]);
  const TetGeom &gt = tg[T];
  const TetGeom &gs = tg[S];
  Moments M;
  moments_zero(M);
  {
    // (lanes of q >= 14 go along with the last point at weight zero)
    const int qq = min(q, 13);
    double r[3], u[3];
    for (int d = 0; d < 3; ++d) {
      double s = 0;
      for (int k = 0; k < 4; ++k) s = fma(qr->tet14[qq][k], gt.v[k][d], s);
      r[d] = s;
      u[d] = s - gt.c[d];
    }
    const double w = q < 14 ? qr->w14[qq] * gt.vol : 0.0;
    dz s0 = mk(0, 0), s1[3] = {mk(0, 0), mk(0, 0), mk(0, 0)};
#pragma unroll 1
    for (int b = 0; b < 9; ++b) {
      if (!((mask >> b) & 1)) continue;
      const int m = b / 3 - 1, n = b % 3 - 1;
      const double o[3] = {r[0] + m * P[pk::A], r[1] + n * P[pk::B], r[2]};
      double pot, V1[3];
      tet_potentials_face(gs.v, f, o, pot, V1);
      const dz ph = kInv4Pi * mk(P[pk::PHRE + b], -P[pk::PHIM + b]);  // e^{+j kt.rho}/(4 pi)
      s0 = s0 + pot * ph;
      for (int d = 0; d < 3; ++d) s1[d] = s1[d] + (V1[d] + (o[d] - gs.c[d]) * pot) * ph;
    }
    double sep[1][3], up[3];
    for (int d = 0; d < 3; ++d) {
      double t = 0;
      for (int k = 0; k < 4; ++k) t = fma(qr->tet4[f][k], gs.v[k][d], t);
      up[d] = t - gs.c[d];
      sep[0][d] = r[d] - t;
    }
    dz g[1];
    pgf_eval_w<true, 1>(P, sep, mask, g);
    const double wq = 0.25 * gs.vol;
    axpy(s0, wq, g[0]);
    for (int d = 0; d < 3; ++d) axpy(s1[d], wq * up[d], g[0]);
    axpy(M.m0, w, s0);
    for (int d = 0; d < 3; ++d) {
      axpy(M.mu[d], w * u[d], s0);
      axpy(M.mv[d], w, s1[d]);
    }
    dz us = mk(0, 0);
    for (int d = 0; d < 3; ++d) axpy(us, u[d], s1[d]);
    axpy(M.muv, w, us);
  }
  // sum the wave (fixed order: deterministic)
  M.m0 = wave_sum64(M.m0);
  M.muv = wave_sum64(M.muv);
  for (int d = 0; d < 3; ++d) {
    M.mu[d] = wave_sum64(M.mu[d]);
    M.mv[d] = wave_sum64(M.mv[d]);
  }
  if (lane >= 16) return;
  const int k = lane >> 2, l = lane & 3;
  scatter_tt_row(M, gt, gs, t2f, T, S, k, l, 1, alpha, gsrc, kappa, k0sq9, out, false, true);
  if (T == S) {
    // mass <f_m, f_n / eps_r>: alpha_k gsrc_l / (9 eps) int_T (r - v_k).(r - v_l), 4-point rule (exact)
    const dz ie = inv_eps[T];
    double s = 0;
    for (int p = 0; p < 4; ++p) {
      double a2 = 0;
      for (int d = 0; d < 3; ++d) {
        double r = 0;
        for (int kk = 0; kk < 4; ++kk) r = fma(qr->tet4[p][kk], gt.v[kk][d], r);
        a2 = fma(r - gt.v[k][d], r - gt.v[l][d], a2);
      }
      s = fma(0.25 * gt.vol, a2, s);
    }
    zput(out, t2f[4 * T + k].unknown, t2f[4 * T + l].unknown, (s / 9.0) * ((alpha[4 * T + k] * gsrc[4 * T + l]) * ie), true);
  }
}

__global__ __launch_bounds__(256) void k_tt_near(const double *__restrict__ pack, int packlen, const QuadRules *__restrict__ qr,
                                                 const TetGeom *__restrict__ tg, const TetFace *__restrict__ t2f,
                                                 const int32_t *__restrict__ lt, const int32_t *__restrict__ ls,
                                                 const int32_t *__restrict__ lmask, int npairs,
                                                 const dz *__restrict__ alpha, const dz *__restrict__ gsrc,
                                                 const dz *__restrict__ kappa, const dz *__restrict__ inv_eps,
                                                 double k0sq9, ZOut out) {
  k_tt_near_body(pack, packlen, qr, tg, t2f, lt, ls, lmask, npairs, alpha, gsrc, kappa, inv_eps, k0sq9, out, blockIdx.x, blockIdx.y);
}

// ------------------------------------------------------------ pairs with faces
// Far rule over (tet, face), 4 x 3 points: M0 = II g_p with the separation
// tet point - face point (DIR = 1) or face point - tet point (DIR = -1), four
// lanes per pair, lane i the tet point i with the three face points; returned
// in every lane of the quad.  REV: also the value of the reversed separations
// (see pgf_eval_w).
template <bool REV, int DIR>
__device__ __forceinline__ void far_tet_face(const double *__restrict__ P, const QuadRules *__restrict__ qr,
                                             const TetGeom &gt, const FaceGeom &f, int i, dz &m0, dz &m0r) {
  double sep[3][3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    double s = 0;
    for (int k = 0; k < 4; ++k) s = fma(qr->tet4[i][k], gt.v[k][d], s);
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const double fp = qr->tri3[j][0] * f.v[0][d] + qr->tri3[j][1] * f.v[1][d] + qr->tri3[j][2] * f.v[2][d];
      sep[j][d] = DIR > 0 ? s - fp : fp - s;
    }
  }
  const double w = 0.25 * gt.vol * (f.area / 3.0);
  dz g[3], gr[3];
  pgf_eval_w<false, 3, REV>(P, sep, 0, g, gr);
  m0 = w * quad_sum(g[0] + g[1] + g[2]);
  if (REV) m0r = w * quad_sum(gr[0] + gr[1] + gr[2]);
}

// test tet (colour class list) x surface-charge face: Z[m_k(T), n_F] -= alpha_Tk sigma_F M0.
// Far pairs only: the touching ones come from the host list (k_tet_face_near).
// The far rules of the two face kernels take the same 4 x 3 point pairs with
// the same weights, so the (tet T, face F) evaluation also gives the value
// M0' of (F as a half-SWG test face, T as source): at normal incidence
// (swap 1) the lattice sum is even and M0' = M0; at oblique incidence
// (swap 2) M0' comes from the reversed-separation form of the same lattice
// sum.  With swap set, each far pair with a half-SWG face writes that entry
// too, Z[m_F, n_l(T)] -= gsrc_Tl kappa_T M0', at the transposed position of
// outT (rows of T's unknowns, columns of faces: the same conflict-free
// pattern as the tet-face entries); the staging copy is added transposed
// after the fill's other kernels.  A wave takes one test tet and 16 faces, and
// lane k of a quad writes the entry of the tet's face k.
template <bool REV>
__device__ __forceinline__ void k_tet_face_body(const double *__restrict__ pack, int packlen, const QuadRules *__restrict__ qr,
                                                  const TetGeom *__restrict__ tg, const TetFace *__restrict__ t2f,
                                                  const int32_t *__restrict__ test_list, int ntest,
                                                  const FaceGeom *__restrict__ fg, int nface,
                                                  const dz *__restrict__ alpha, const dz *__restrict__ sigma,
                                                  const dz *__restrict__ gsrc, const dz *__restrict__ kappa,
                                                  ZOut out, ZOut outT, int swap, int bx_, int by_) {
  extern __shared__ double s_tab[];
  stage_table(pack, packlen, s_tab);
  const int ti = uniform(by_ * 4 + (threadIdx.x >> 6));
  const int fi = bx_ * 16 + ((threadIdx.x & 63) >> 2), k = threadIdx.x & 3;
  if (ti >= ntest || fi >= nface) return;
  const int T = uniform(test_list[ti]);
  const TetGeom &gt = tg[T];
  const FaceGeom &f = fg[fi];
  if (touch_mask(gt.canon, gt.off, 4, f.canon, f.off, 3)) return;
  dz m0, m0r;
  far_tet_face<REV, 1>(s_tab, qr, gt, f, k, m0, m0r);
  if (!REV) m0r = m0;
  const int64_t row = t2f[4 * T + k].unknown;
  zput(out, row, f.unknown, mk(0, 0) - alpha[4 * T + k] * (sigma[fi] * m0), false);
  if (swap && f.half) zput(outT, row, f.unknown, mk(0, 0) - gsrc[4 * T + k] * (m0r * kappa[T]), false);
}

__global__ __launch_bounds__(256, 2) void k_tet_face(const double *__restrict__ pack, int packlen, const QuadRules *__restrict__ qr,
                                                  const TetGeom *__restrict__ tg, const TetFace *__restrict__ t2f,
                                                  const int32_t *__restrict__ test_list, int ntest,
                                                  const FaceGeom *__restrict__ fg, int nface,
                                                  const dz *__restrict__ alpha, const dz *__restrict__ sigma,
                                                  const dz *__restrict__ gsrc, const dz *__restrict__ kappa,
                                                  ZOut out, ZOut outT, int swap) {
  k_tet_face_body<false>(pack, packlen, qr, tg, t2f, test_list, ntest, fg, nface, alpha, sigma, gsrc, kappa, out, outT,
                         swap == 2 ? 0 : swap, blockIdx.x, blockIdx.y);
}
// oblique incidence with the staging copy: the (face, tet) entries from the
// reversed separation (swap 2); a kernel of its own, whose registers the
// two-separation form does not take from k_tet_face
__global__ __launch_bounds__(256, 2) void k_tet_face_rev(const double *__restrict__ pack, int packlen,
                                                      const QuadRules *__restrict__ qr, const TetGeom *__restrict__ tg,
                                                      const TetFace *__restrict__ t2f,
                                                      const int32_t *__restrict__ test_list, int ntest,
                                                      const FaceGeom *__restrict__ fg, int nface,
                                                      const dz *__restrict__ alpha, const dz *__restrict__ sigma,
                                                      const dz *__restrict__ gsrc, const dz *__restrict__ kappa,
                                                      ZOut out, ZOut outT) {
  k_tet_face_body<true>(pack, packlen, qr, tg, t2f, test_list, ntest, fg, nface, alpha, sigma, gsrc, kappa, out, outT, 2,
                        blockIdx.x, blockIdx.y);
}

// Touching (test tet, surface-charge face) pairs of one test colour: outer
// 14-point rule on T, closed-form int_F 1/R per touching image, 3-point inner
// rule for the remainder.  16 lanes per pair, lane q < 14 the outer point q;
// lane k < 4 writes the entry of the tet's face k.  (One lane per pair took
// 1.0 ms per launch whatever the size, four launches per fill.)
__device__ __forceinline__ void k_tet_face_near_body(const double *__restrict__ pack, int packlen,
                                                       const QuadRules *__restrict__ qr, const TetGeom *__restrict__ tg,
                                                       const TetFace *__restrict__ t2f, const int32_t *__restrict__ pairs,
                                                       int npairs, const FaceGeom *__restrict__ fg,
                                                       const dz *__restrict__ alpha, const dz *__restrict__ sigma,
                                                       ZOut out, int bx_, int by_) {
  extern __shared__ double s_tab[];
  stage_table(pack, packlen, s_tab);
  const double *__restrict__ P = s_tab;
  const int q = threadIdx.x & 15, i = bx_ * 16 + (threadIdx.x >> 4);
  // (lanes past the last pair or point go along at weight zero: the sums below take whole waves)
  const int ii = min(i, npairs - 1), qq = min(q, 13);
  const int T = pairs[2 * ii], fi = pairs[2 * ii + 1];
  const TetGeom &gt = tg[T];
  const FaceGeom &f = fg[fi];
  const int mask = touch_mask(gt.canon, gt.off, 4, f.canon, f.off, 3);
  double r[3];
  for (int d = 0; d < 3; ++d) {
    double s = 0;
    for (int k = 0; k < 4; ++k) s = fma(qr->tet14[qq][k], gt.v[k][d], s);
    r[d] = s;
  }
  dz s0 = mk(0, 0);
#pragma unroll 1
  for (int b = 0; b < 9; ++b) {
    if (!((mask >> b) & 1)) continue;
    const int m = b / 3 - 1, n = b % 3 - 1;
    const double o[3] = {r[0] + m * P[pk::A], r[1] + n * P[pk::B], r[2]};
    double iinv, ione;
    tri_potentials(f.v[0], f.v[1], f.v[2], o, iinv, ione);
    s0 = s0 + (kInv4Pi * iinv) * mk(P[pk::PHRE + b], -P[pk::PHIM + b]);
  }
#pragma unroll 1
  for (int j = 0; j < 3; ++j) {
    double sep[1][3];
    for (int d = 0; d < 3; ++d)
      sep[0][d] = r[d] - (qr->tri3[j][0] * f.v[0][d] + qr->tri3[j][1] * f.v[1][d] + qr->tri3[j][2] * f.v[2][d]);
    dz g[1];
    pgf_eval_w<true, 1>(P, sep, mask, g);
    axpy(s0, f.area / 3.0, g[0]);
  }
  const dz m0 = dpp_add<0x140>(mirror8_sum(quad_sum((q < 14 ? qr->w14[qq] * gt.vol : 0.0) * s0)));
  if (i >= npairs || q >= 4) return;
  zput(out, t2f[4 * T + q].unknown, f.unknown, mk(0, 0) - alpha[4 * T + q] * (sigma[fi] * m0), true);
}

__global__ __launch_bounds__(256, 2) void k_tet_face_near(const double *__restrict__ pack, int packlen,
                                                       const QuadRules *__restrict__ qr, const TetGeom *__restrict__ tg,
                                                       const TetFace *__restrict__ t2f, const int32_t *__restrict__ pairs,
                                                       int npairs, const FaceGeom *__restrict__ fg,
                                                       const dz *__restrict__ alpha, const dz *__restrict__ sigma,
                                                       ZOut out) {
  k_tet_face_near_body(pack, packlen, qr, tg, t2f, pairs, npairs, fg, alpha, sigma, out, blockIdx.x, blockIdx.y);
}

// half-SWG test face x source tet (colour class list): Z[m_F, n_l(S)] -= gsrc_Sl kappa_S M0.
// Far pairs only: the touching ones come from the host list (k_face_tet_near).
// A wave takes one face and 16 tets; lane l of a quad writes the entry of the
// tet's face l.
__device__ __forceinline__ void k_face_tet_body(const double *__restrict__ pack, int packlen, const QuadRules *__restrict__ qr,
                                                  const FaceGeom *__restrict__ fg, const int32_t *__restrict__ half_list,
                                                  int nhalf, const TetGeom *__restrict__ tg,
                                                  const TetFace *__restrict__ t2f, const int32_t *__restrict__ src_list,
                                                  int nsrc, const dz *__restrict__ gsrc, const dz *__restrict__ kappa,
                                                  ZOut out, int bx_, int by_) {
  extern __shared__ double s_tab[];
  stage_table(pack, packlen, s_tab);
  const int hi = uniform(by_ * 4 + (threadIdx.x >> 6));
  const int si = bx_ * 16 + ((threadIdx.x & 63) >> 2), l = threadIdx.x & 3;
  if (hi >= nhalf || si >= nsrc) return;
  const FaceGeom &f = fg[uniform(half_list[hi])];
  const int S = src_list[si];
  const TetGeom &gs = tg[S];
  if (touch_mask(f.canon, f.off, 3, gs.canon, gs.off, 4)) return;
  dz m0, unused;
  far_tet_face<false, -1>(s_tab, qr, gs, f, l, m0, unused);
  zput(out, f.unknown, t2f[4 * S + l].unknown, mk(0, 0) - gsrc[4 * S + l] * (m0 * kappa[S]), false);
}

__global__ __launch_bounds__(256, 2) void k_face_tet(const double *__restrict__ pack, int packlen, const QuadRules *__restrict__ qr,
                                                  const FaceGeom *__restrict__ fg, const int32_t *__restrict__ half_list,
                                                  int nhalf, const TetGeom *__restrict__ tg,
                                                  const TetFace *__restrict__ t2f, const int32_t *__restrict__ src_list,
                                                  int nsrc, const dz *__restrict__ gsrc, const dz *__restrict__ kappa,
                                                  ZOut out) {
  k_face_tet_body(pack, packlen, qr, fg, half_list, nhalf, tg, t2f, src_list, nsrc, gsrc, kappa, out, blockIdx.x, blockIdx.y);
}

// Touching (half-SWG test face, source tet) pairs of one source colour: outer
// 7-point rule on F, closed-form int_S 1/R, 4-point inner rule for the
// remainder.  32 lanes per pair, lane 4 p + c the outer point p < 7 with the
// face c of S in the closed form and the inner point c in the remainder.
__device__ __forceinline__ void k_face_tet_near_body(const double *__restrict__ pack, int packlen,
                                                       const QuadRules *__restrict__ qr, const FaceGeom *__restrict__ fg,
                                                       const int32_t *__restrict__ half_list,
                                                       const TetGeom *__restrict__ tg, const TetFace *__restrict__ t2f,
                                                       const int32_t *__restrict__ pairs, int npairs,
                                                       const dz *__restrict__ gsrc, const dz *__restrict__ kappa,
                                                       ZOut out, int bx_, int by_) {
  extern __shared__ double s_tab[];
  stage_table(pack, packlen, s_tab);
  const double *__restrict__ P = s_tab;
  const int i = bx_ * 8 + (threadIdx.x >> 5), p = (threadIdx.x & 31) >> 2, c = threadIdx.x & 3;
  const int ii = min(i, npairs - 1), pp = min(p, 6);   // (lanes past the last pair or point: weight zero)
  const int hi = pairs[2 * ii], S = pairs[2 * ii + 1];
  const FaceGeom &f = fg[half_list[hi]];
  const TetGeom &gs = tg[S];
  const int mask = touch_mask(f.canon, f.off, 3, gs.canon, gs.off, 4);
  double r[3], sep[1][3];
  for (int d = 0; d < 3; ++d) {
    r[d] = qr->tri7[pp][0] * f.v[0][d] + qr->tri7[pp][1] * f.v[1][d] + qr->tri7[pp][2] * f.v[2][d];
    double s = 0;
    for (int k = 0; k < 4; ++k) s = fma(qr->tet4[c][k], gs.v[k][d], s);
    sep[0][d] = r[d] - s;
  }
  dz s0 = mk(0, 0);
#pragma unroll 1
  for (int b = 0; b < 9; ++b) {
    if (!((mask >> b) & 1)) continue;
    const int m = b / 3 - 1, n = b % 3 - 1;
    const double o[3] = {r[0] + m * P[pk::A], r[1] + n * P[pk::B], r[2]};
    double pot, V1[3];
    tet_potentials_face(gs.v, c, o, pot, V1);
    s0 = s0 + (kInv4Pi * pot) * mk(P[pk::PHRE + b], -P[pk::PHIM + b]);
  }
  dz g[1];
  pgf_eval_w<true, 1>(P, sep, mask, g);
  axpy(s0, 0.25 * gs.vol, g[0]);
  dz m0 = dpp_add<0x140>(mirror8_sum(quad_sum((p < 7 ? qr->w7[pp] * f.area : 0.0) * s0)));
  m0 = mk(m0.re + __shfl_xor(m0.re, 16), m0.im + __shfl_xor(m0.im, 16)) * kappa[S];
  if (i >= npairs || p > 0) return;
  zput(out, f.unknown, t2f[4 * S + c].unknown, mk(0, 0) - gsrc[4 * S + c] * m0, true);
}

__global__ __launch_bounds__(256, 2) void k_face_tet_near(const double *__restrict__ pack, int packlen,
                                                       const QuadRules *__restrict__ qr, const FaceGeom *__restrict__ fg,
                                                       const int32_t *__restrict__ half_list,
                                                       const TetGeom *__restrict__ tg, const TetFace *__restrict__ t2f,
                                                       const int32_t *__restrict__ pairs, int npairs,
                                                       const dz *__restrict__ gsrc, const dz *__restrict__ kappa,
                                                       ZOut out) {
  k_face_tet_near_body(pack, packlen, qr, fg, half_list, tg, t2f, pairs, npairs, gsrc, kappa, out, blockIdx.x, blockIdx.y);
}

// half-SWG test face x surface-charge face: Z[m_F, n_G] += sigma_G M0.  A wave
// takes one test face and kFaceChunk = 21 source faces, three lanes each: first
// the far pairs, lane 3 s + i the point i of the test face with the source
// face's three points (none with no dense part in the destination, the
// structured-grid operator, whose far pairs come from its FFT tables), then
// the few touching ones, three at a time: outer 7-point rule, lane 21 s + 3 p +
// j the outer point p of the s-th pair and the inner point j of the 3-point
// rule for the remainder, the closed form int_G 1/R with j = 0.  On small cells
// one wave's chain is the launch: N = 416, 122 us (199 with 64 source faces
// per wave, the points of a far pair in turn).
__device__ __forceinline__ void k_face_face_body(const double *__restrict__ pack, int packlen, const QuadRules *__restrict__ qr,
                                                   const FaceGeom *__restrict__ fg,
                                                   const int32_t *__restrict__ half_list, int nhalf, int nface,
                                                   const dz *__restrict__ sigma, ZOut out, int bx_, int by_) {
  extern __shared__ double s_tab[];
  __shared__ dz parts[4][64];
  stage_table(pack, packlen, s_tab);
  const double *__restrict__ P = s_tab;

  const int lane = threadIdx.x & 63, ls = lane / 3, li = lane - 3 * ls;   // (lane 63: ls = 21, idle)
  const int hi = uniform(by_ * 4 + (threadIdx.x >> 6));
  const int gi = bx_ * kFaceChunk + ls;
  if (hi >= nhalf) return;
  const FaceGeom &f = fg[uniform(half_list[hi])];
  const FaceGeom &gl = fg[min(gi, nface - 1)];
  const bool ok = ls < kFaceChunk && gi < nface;
  const int mask = ok ? touch_mask(f.canon, f.off, 3, gl.canon, gl.off, 3) : 0;
  if (out.Z || out.Zs) {
    dz acc = mk(0, 0);
    if (ok && mask == 0) {
      double sep[3][3];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const double r = qr->tri3[li][0] * f.v[0][d] + qr->tri3[li][1] * f.v[1][d] + qr->tri3[li][2] * f.v[2][d];
#pragma unroll
        for (int j = 0; j < 3; ++j)
          sep[j][d] = r - (qr->tri3[j][0] * gl.v[0][d] + qr->tri3[j][1] * gl.v[1][d] + qr->tri3[j][2] * gl.v[2][d]);
      }
      dz g[3];
      pgf_eval_w<false, 3>(P, sep, 0, g);
      acc = g[0] + g[1] + g[2];
    }
    const dz a1 = mk(__shfl_down(acc.re, 1), __shfl_down(acc.im, 1)), a2 = mk(__shfl_down(acc.re, 2), __shfl_down(acc.im, 2));
    acc = (acc + a1) + a2;
    if (ok && mask == 0 && li == 0)
      zput(out, f.unknown, gl.unknown, sigma[gi] * ((f.area / 3.0 * (gl.area / 3.0)) * acc), false);
  }
  const int s3 = min(lane / 21, 2), p = (lane - 21 * s3) / 3, j = (lane - 21 * s3) % 3;   // (lane 63: p = 7, idle)
  for (unsigned long long todo = __ballot(mask != 0 && li == 0); todo != 0;) {
    // the next three touching faces' lanes (fewer at the end: the last one again, not stored)
    int src[3], np = 0;
    for (int s = 0; s < 3; ++s) {
      if (todo != 0) {
        src[s] = __ffsll((long long)todo) - 1;
        todo &= todo - 1;
        np = s + 1;
      } else {
        src[s] = src[np - 1];
      }
    }
    const int mine = s3 == 0 ? src[0] : (s3 == 1 ? src[1] : src[2]);
    const int tm = __shfl(mask, mine), ti = bx_ * kFaceChunk + mine / 3;
    const FaceGeom &g = fg[ti];
    const int pp = min(p, 6);
    double r[3], sep[1][3];
    for (int d = 0; d < 3; ++d) {
      r[d] = qr->tri7[pp][0] * f.v[0][d] + qr->tri7[pp][1] * f.v[1][d] + qr->tri7[pp][2] * f.v[2][d];
      sep[0][d] = r[d] - (qr->tri3[j][0] * g.v[0][d] + qr->tri3[j][1] * g.v[1][d] + qr->tri3[j][2] * g.v[2][d]);
    }
    dz s0 = mk(0, 0);
#pragma unroll 1
    for (int b = 0; b < 9; ++b) {
      if (!((tm >> b) & 1)) continue;
      const int m = b / 3 - 1, n = b % 3 - 1;
      const double o[3] = {r[0] + m * P[pk::A], r[1] + n * P[pk::B], r[2]};
      double iinv, ione;
      tri_potentials(g.v[0], g.v[1], g.v[2], o, iinv, ione);
      if (j == 0) s0 = s0 + (kInv4Pi * iinv) * mk(P[pk::PHRE + b], -P[pk::PHIM + b]);
    }
    dz gv[1];
    pgf_eval_w<true, 1>(P, sep, tm, gv);
    axpy(s0, g.area / 3.0, gv[0]);
    dz *part = parts[threadIdx.x >> 6];   // this wave's 64 slots
    part[lane] = (p < 7 ? qr->w7[pp] * f.area : 0.0) * s0;
    __builtin_amdgcn_wave_barrier();
    if (p == 0 && j == 0 && s3 < np) {
      dz m0 = mk(0, 0);
      for (int e = 0; e < 21; ++e) m0 = m0 + part[21 * s3 + e];
      zput(out, f.unknown, g.unknown, sigma[ti] * m0, true);
    }
    __builtin_amdgcn_wave_barrier();
  }
}

__global__ __launch_bounds__(256, 2) void k_face_face(const double *__restrict__ pack, int packlen, const QuadRules *__restrict__ qr,
                                                   const FaceGeom *__restrict__ fg,
                                                   const int32_t *__restrict__ half_list, int nhalf, int nface,
                                                   const dz *__restrict__ sigma, ZOut out) {
  k_face_face_body(pack, packlen, qr, fg, half_list, nhalf, nface, sigma, out, blockIdx.x, blockIdx.y);
}

// ------------------------------------------------------------ fused multi-cell fill
__global__ __launch_bounds__(256, kFarWaves) void k_tt_far_seg(const FarSeg *__restrict__ segs, int nseg) {
  VIE_SEG_BEGIN(FarSeg)
  tt_far_body<false>(A.pack, A.packlen, A.qr, A.tg, A.t2f, A.test_list, A.ntest, A.src_list, A.nsrc, A.alpha, A.gsrc,
                     A.kappa, A.k0sq9, A.out, A.outT, A.sym, A.tper, bx, by);
}
__global__ __launch_bounds__(256, kFarWaves) void k_tt_far_rev_seg(const FarSeg *__restrict__ segs, int nseg) {
  VIE_SEG_BEGIN(FarSeg)
  tt_far_body<true>(A.pack, A.packlen, A.qr, A.tg, A.t2f, A.test_list, A.ntest, A.src_list, A.nsrc, A.alpha, A.gsrc,
                    A.kappa, A.k0sq9, A.out, A.outT, A.sym, A.tper, bx, by);
}
__global__ __launch_bounds__(256) void k_tt_near_seg(const NearSeg *__restrict__ segs, int nseg) {
  VIE_SEG_BEGIN(NearSeg)
  k_tt_near_body(A.pack, A.packlen, A.qr, A.tg, A.t2f, A.lt, A.ls, A.lmask, A.npairs, A.alpha, A.gsrc, A.kappa,
                 A.inv_eps, A.k0sq9, A.out, bx, by);
}
__global__ __launch_bounds__(256, 2) void k_tet_face_seg(const TetFaceSeg *__restrict__ segs, int nseg) {
  VIE_SEG_BEGIN(TetFaceSeg)
  k_tet_face_body<false>(A.pack, A.packlen, A.qr, A.tg, A.t2f, A.test_list, A.ntest, A.fg, A.nface, A.alpha, A.sigma,
                         A.gsrc, A.kappa, A.out, A.outT, A.swap, bx, by);
}
__global__ __launch_bounds__(256, 2) void k_tet_face_rev_seg(const TetFaceSeg *__restrict__ segs, int nseg) {
  VIE_SEG_BEGIN(TetFaceSeg)
  k_tet_face_body<true>(A.pack, A.packlen, A.qr, A.tg, A.t2f, A.test_list, A.ntest, A.fg, A.nface, A.alpha, A.sigma,
                        A.gsrc, A.kappa, A.out, A.outT, A.swap, bx, by);
}
__global__ __launch_bounds__(256, 2) void k_tet_face_near_seg(const TetFaceNearSeg *__restrict__ segs, int nseg) {
  VIE_SEG_BEGIN(TetFaceNearSeg)
  k_tet_face_near_body(A.pack, A.packlen, A.qr, A.tg, A.t2f, A.pairs, A.npairs, A.fg, A.alpha, A.sigma, A.out, bx, by);
}
__global__ __launch_bounds__(256, 2) void k_face_tet_seg(const FaceTetSeg *__restrict__ segs, int nseg) {
  VIE_SEG_BEGIN(FaceTetSeg)
  k_face_tet_body(A.pack, A.packlen, A.qr, A.fg, A.half_list, A.nhalf, A.tg, A.t2f, A.src_list, A.nsrc, A.gsrc,
                  A.kappa, A.out, bx, by);
}
__global__ __launch_bounds__(256, 2) void k_face_tet_near_seg(const FaceTetNearSeg *__restrict__ segs, int nseg) {
  VIE_SEG_BEGIN(FaceTetNearSeg)
  k_face_tet_near_body(A.pack, A.packlen, A.qr, A.fg, A.half_list, A.tg, A.t2f, A.pairs, A.npairs, A.gsrc, A.kappa,
                       A.out, bx, by);
}
__global__ __launch_bounds__(256, 2) void k_face_face_seg(const FaceFaceSeg *__restrict__ segs, int nseg) {
  VIE_SEG_BEGIN(FaceFaceSeg)
  k_face_face_body(A.pack, A.packlen, A.qr, A.fg, A.half_list, A.nhalf, A.nface, A.sigma, A.out, bx, by);
}

// ------------------------------------------------------------ right-hand side
// b_m = sum_{T in m} chi s a_m/(3 V_T) int_T (r - p).E^i dV, 14-point rule;
// one thread per unknown (gathers its two halves, no write conflicts).
__global__ void k_rhs(int64_t N, const int32_t *__restrict__ utet, const int32_t *__restrict__ uk,
                      const TetGeom *__restrict__ tg, const QuadRules *__restrict__ qr, const dz *__restrict__ alpha,
                      double kix, double kiy, double kiz, double ex, double ey, double ez, dz *__restrict__ b) {
  const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= N) return;
  dz acc = mk(0, 0);
  for (int h = 0; h < 2; ++h) {
    const int T = utet[2 * m + h];
    if (T < 0) continue;
    const int k = uk[2 * m + h];
    const TetGeom &g = tg[T];
    dz s = mk(0, 0);
    for (int q = 0; q < 14; ++q) {
      double r[3];
      for (int d = 0; d < 3; ++d) {
        double t = 0;
        for (int kk = 0; kk < 4; ++kk) t = fma(qr->tet14[q][kk], g.v[kk][d], t);
        r[d] = t;
      }
      const double proj = (r[0] - g.v[k][0]) * ex + (r[1] - g.v[k][1]) * ey + (r[2] - g.v[k][2]) * ez;
      double sn, cs;
      sincos(-(kix * r[0] + kiy * r[1] + kiz * r[2]), &sn, &cs);
      axpy(s, qr->w14[q] * g.vol * proj, mk(cs, sn));
    }
    acc = acc + alpha[4 * T + k] * ((1.0 / 3.0) * s);
  }
  b[m] = acc;
}

// ------------------------------------------------------------ diagnostics
__global__ void k_pgf_probe(const double *__restrict__ pack, int packlen, const double *__restrict__ d, int64_t n,
                            dz *__restrict__ out) {
  extern __shared__ double s_tab[];
  stage_table(pack, packlen, s_tab);
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  out[i] = pgf_eval<false>(s_tab, d[3 * i], d[3 * i + 1], d[3 * i + 2], 0);
}

// gather Z entries (mixed precision: FP32 far part plus the FP64 near entry)
__global__ void k_gather(ZOut Z, const int64_t *__restrict__ rows, const int64_t *__restrict__ cols, int64_t k,
                         dz *__restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= k) return;
  const int64_t m = rows[i], n = cols[i];
  if (Z.Z) {
    out[i] = Z.Z[m * Z.ld + n];
    return;
  }
  const fz f = Z.Zs[m * Z.ld + n];
  dz v = mk(f.re, f.im);
  int64_t lo = Z.rowptr[m], hi = Z.rowptr[m + 1];
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (Z.cols[mid] < n) lo = mid + 1;
    else hi = mid;
  }
  if (lo < Z.rowptr[m + 1] && Z.cols[lo] == n) v = v + Z.vals[lo];
  out[i] = v;
}

}  // namespace vie
