// Device code shared by the fill kernels: the store into Z, moments of a
// tetrahedron pair, and the segments of the fused multi-cell launches.
#pragma once
#include <hip/hip_runtime.h>

#include "kernels.h"

namespace vie {

static constexpr double kInv4Pi = 0.079577471545947667884;

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Z[m][n] += v into the destination of this fill (see ZOut).  In mixed
// precision a far contribution is added to the FP32 entry in FP64 and rounded
// once; a near one goes to its slot of the sorted CSR row.
__device__ __forceinline__ void zput(const ZOut &o, int64_t m, int64_t n, dz v, bool near) {
  if (o.Z) {
    dz *p = o.Z + m * o.ld + n;
    *p = *p + v;
  } else if (near) {
    int64_t lo = o.rowptr[m], hi = o.rowptr[m + 1];
    while (lo < hi) {
      const int64_t mid = (lo + hi) >> 1;
      if (o.cols[mid] < n) lo = mid + 1;
      else hi = mid;
    }
    if (lo < o.rowptr[m + 1] && o.cols[lo] == n) o.vals[lo] = o.vals[lo] + v;
  } else {
    fz *p = o.Zs + m * o.ld + n;
    const fz z = *p;
    *p = fz{(float)((double)z.re + v.re), (float)((double)z.im + v.im)};
  }
}

// ------------------------------------------------------------ tet-pair moments
struct Moments {
  dz m0, mu[3], mv[3], muv;
};

__device__ __forceinline__ void moments_zero(Moments &M) {
  M.m0 = mk(0, 0);
  M.muv = mk(0, 0);
  for (int d = 0; d < 3; ++d) M.mu[d] = M.mv[d] = mk(0, 0);
}

// The segment of fused-grid block b (segments ordered by their first block).
template <class S>
__device__ __forceinline__ int seg_of(const S *__restrict__ segs, int nseg, int b) {
  int lo = 0, hi = nseg - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (segs[mid].first <= b) lo = mid;
    else hi = mid - 1;
  }
  return uniform(lo);
}

#define VIE_SEG_BEGIN(S)                                  \
  const int s_ = seg_of(segs, nseg, (int)blockIdx.x);     \
  const S &A = segs[s_];                                  \
  const int lb_ = (int)blockIdx.x - A.first;              \
  const int bx = lb_ % A.gx, by = lb_ / A.gx;

}  // namespace vie
