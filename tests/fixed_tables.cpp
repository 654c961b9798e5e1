// Digest of the lattice-sum coefficients that the mixed-precision operator
// holds to: one line per cell and incidence given on stdin ("a b zspan lambda
// theta phi"), the FNV-1a hash of every kept coefficient and degree.
#include <cstdio>
#include <cstring>
#include <memory>

#include "host.h"

static uint64_t hash = 0;
static void add(const void *p, size_t n) {
  for (size_t i = 0; i < n; ++i) hash = (hash ^ ((const unsigned char *)p)[i]) * 1099511628211ull;
}

int main() {
  auto tab = std::make_unique<vie::PgfTable>();
  double a, b, z, lam, th, ph, margin;
  while (std::scanf("%lf %lf %lf %lf %lf %lf", &a, &b, &z, &lam, &th, &ph) == 6) {
    const std::string e = vie::build_pgf_table(*tab, a, b, z, lam, th, ph, &margin, vie::PgfTerms::fixed);
    if (!e.empty() || margin < 0.02) return 1;
    hash = 14695981039346656037ull;
    for (int i = 0; i < tab->nimg; ++i) {
      const vie::PgfImage &im = tab->img[i];
      add(&im.deg, 4);
      add(im.f, 8 * (size_t)(im.deg + 1));
      add(&im.hdeg, 4);
      if (im.hdeg >= 0) add(im.h, 8 * (size_t)(im.hdeg + 1));
    }
    for (const vie::PgfMode &md : tab->mode) {
      add(&md.deg, 4);
      if (md.deg < 0) continue;
      add(md.kre, 8 * (size_t)(md.deg + 1));
      if (md.cplx) add(md.kim, 8 * (size_t)(md.deg + 1));
    }
    std::printf("%016llx\n", (unsigned long long)hash);
  }
  return 0;
}
