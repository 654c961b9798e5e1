// Host-side internals of libvie: mesh topology, quadrature rules, lattice-sum
// tables and the special functions used to build them.
#pragma once
#include <complex>
#include <string>
#include <vector>

#include "common.h"

namespace vie {

using zd = std::complex<double>;

struct MeshTopology {
  double a = 0, b = 0;
  int64_t nv = 0, nt = 0;
  int ndom = 0;
  std::vector<double> verts;        // 3*nv
  std::vector<int32_t> tets;        // 4*nt
  std::vector<int32_t> dom;         // nt
  std::vector<int32_t> canon;       // nv  canonical vertex id
  std::vector<int32_t> offx, offy;  // nv  lattice offset of each vertex
  std::vector<double> vol;          // nt
  double zmin = 0, zmax = 0;
  double max_diam = 0;              // largest tetrahedron diameter

  int64_t N = 0;                    // unknowns
  std::vector<int32_t> face_vid;    // 3N (as the face sits in T+)
  std::vector<int32_t> tplus, tminus, fdom, freep, freem;
  std::vector<int32_t> shx, shy;    // lattice shift of T-'s copy
  std::vector<double> area;         // N
  std::vector<TetFace> t2f;         // 4*nt
  std::vector<int32_t> charged;     // surface-charge faces (unknown ids), increasing
  std::vector<int64_t> dstart, dend;

  // conflict-free colouring of the tetrahedra (face-adjacent tets differ)
  int ncolors = 0;
  std::vector<int32_t> color;                     // nt
  std::vector<std::vector<int32_t>> color_tets;   // per colour, increasing
  // touching tet pairs, grouped by (colour(T), colour(T')): test, source, image mask
  std::vector<std::vector<int32_t>> near_t, near_s, near_mask;
  // touching (tet T, surface-charge face) pairs grouped by colour(T): T and the
  // face's position in `charged`, interleaved
  std::vector<std::vector<int32_t>> near_tf;
  // touching (half-SWG face, tet S) pairs grouped by colour(S): the face's
  // position among the half-SWG faces of `charged`, and S, interleaved
  std::vector<std::vector<int32_t>> near_ft;
};

// Returns "" on success, else an error message.
std::string build_topology(MeshTopology &t, const double *verts, int64_t nv, const int32_t *tets, int64_t nt,
                           const int32_t *tet_domain, int ndom, double a, double b);

// Sparsity pattern of the near (touching-pair) entries of Z, CSR with sorted
// rows (rowptr [N+1], cols [nnz]).
void build_near_pattern(const MeshTopology &t, std::vector<int64_t> &rowptr, std::vector<int32_t> &cols);

// Tetrahedron holding each of n points (3n doubles): the lowest index among
// those whose barycentric coordinates are all >= -1e-12, -1 if none.
void locate_points(const MeshTopology &t, const double *pts, int64_t n, int32_t *tet);

// Touching-image mask (bit (m+1)*3 + (n+1)) of two vertex sets given by canonical
// ids and packed offsets ((ox+2) | (oy+2) << 4).
inline int touching_mask(const int32_t *ct, const int32_t *ot, int nt_, const int32_t *cs, const int32_t *os,
                         int ns) {
  int mask = 0;
  for (int i = 0; i < nt_; ++i)
    for (int j = 0; j < ns; ++j)
      if (ct[i] == cs[j]) {
        int dm = (os[j] & 15) - (ot[i] & 15);
        int dn = (os[j] >> 4) - (ot[i] >> 4);
        mask |= 1 << ((dm + 1) * 3 + (dn + 1));
      }
  return mask;
}

void build_quadrature(QuadRules &q);

// How the fitted functions are evaluated: their expansion in the wavenumber
// (2 ms per table), or the quadratures whose every coefficient the
// mixed-precision operator holds to.
enum class PgfTerms { series, fixed };

// Ewald split and per-fill tables.  zspan = zmax - zmin of the mesh.
// Returns "" or an error; sets *wood_margin = min_{(p,q)!=(0,0)} |gamma_pq|/k0.
std::string build_pgf_table(PgfTable &tab, double a, double b, double zspan, double lambda, double theta,
                            double phi, double *wood_margin, PgfTerms terms = PgfTerms::series);

// Compact copy of the table for the kernels (staged into LDS): only the
// fitted coefficients of the significant terms, in doubles.  A series is
// [K, e_0 .. e_K], its coefficients with the highest degree first, K even
// (a zero e_0 for odd degrees).  Layout:
//   [0..10)  E, a, b, 1/a, 1/b, kx/pi, ky/pi, form (0 monomials, 1 Chebyshev),
//            offset of the order rows (high word: p_lo + 8 | (p_hi + 8) << 8), ws E^2
//   [10..19) Re phase0[9], [19..28) Im phase0[9], [28] offset of the
//            propagating orders (high word: their count)
//   [29..34) per m = 0..4: n_m, the number of image records (m, 0 .. n_m - 1)
//   image records from kPackImages on, rows m in order, each standing for
//     (+-m, +-n): [E xs, -(xa xs + 1), Re, Im phase of (m, n), of (m, -n)],
//     the F series (high word of its K: record length), the H series (m, n <= 1)
//   order rows p = p_hi .. p_lo, each [q_max (high word: has differences), 0],
//     the series of (p, 0), then for q = 1 .. q_max the sum s of those of (p, q)
//     and (p, -q), or if a difference d in the row is not zero both,
//     [K, 0, (s_0, d_0) .. (s_K, d_K)] (real parts)
//   propagating orders, each [p (high word: q), 0] and the series of Im K_pq
// Integers are in the low and high 32 bits of their slots.
constexpr int kPackRows = 29;
constexpr int kPackImages = 40;
void pack_pgf_table(const PgfTable &tab, std::vector<double> &out);

// The copy for the far kernels of the mixed-precision operator (offsets in common.h):
//   [0..10)  E, a, b, 1/a, 1/b, kx, ky, 2pi/a, 2pi/b, ws
//   [10..19) Re phase0[9], [19..28) Im phase0[9], [28] the largest |m| of an
//            image, [29..34) per |m| the largest |n| (every smaller one is there)
//   per row p of the order grid a bit per slot q with an order (high word: of
//            those with an imaginary part)
//   records: the images in the order of (m, n), each [E xs, -(xa xs + 1), Re, Im
//   phase] and the F series, then the orders in the order of (p, q), each its
//   real series and, if it propagates, its imaginary one.  A series is [K, c_K,
//   c_{K-1}, c_{K-2} - c_K, c_{K-3} .. c_0], K even, the record's length in the
//   high word of K; both start at multiples of four.
void pack_pgf_fixed(const PgfTable &tab, std::vector<double> &out);
// Doubles of a table that lists every image and every order by itself, in
// groups of four coefficients.
size_t pgf_listed_doubles(const PgfTable &tab);

}  // namespace vie
