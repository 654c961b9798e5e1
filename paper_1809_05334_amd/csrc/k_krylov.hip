// GMRES building blocks (Sec. 3): dense complex matrix-vector product,
// classical Gram-Schmidt (applied twice) against the Krylov basis, norms,
// Givens rotations on the Hessenberg matrix, and the final small solve.
// All in FP64.
#include <hip/hip_runtime.h>

#include "kernels.h"

namespace vie {

__device__ __forceinline__ dz wsum(dz v) {
  for (int o = 32; o > 0; o >>= 1) {
    v.re += __shfl_xor(v.re, o);
    v.im += __shfl_xor(v.im, o);
  }
  return v;
}
__device__ __forceinline__ double wsum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// y = Z x  (or y = b - Z x when b != nullptr).  Z row-major, N x ld.
// A block of 4 waves owns 4*RPW consecutive rows; x is staged through LDS in
// chunks shared by the block, Z is streamed once with non-temporal loads.
// With NV = 2 one pass over Z serves two vectors (the two polarisations of a
// paired solve); each vector's sums run in the same order as with NV = 1.
// Loads are unconditional (rows past N read row N-1 and are never stored,
// staging reads past the chunk are clamped into it): a load under a branch is
// waited for inside the branch, which would serialise a wave's loads.
constexpr int kMvChunk = 1024;

// x chunk [c0, c0+len) of each vector into xs (vector q at q*kMvChunk):
// every load first, as two-double vectors held in registers (copies of the
// complex struct were kept in scratch memory), then the shared stores
typedef double v2d __attribute__((ext_vector_type(2)));
static_assert(kMvChunk == 4 * 256, "four staging loads per thread and vector");
template <int NV>
__device__ __forceinline__ void stage_x(const MvVecs &v, int64_t c0, int len, dz *xs) {
  static_assert(NV == 1 || NV == 2, "one or two vectors");
  const int tid = threadIdx.x;
  const int i0 = min(tid, len - 1), i1 = min(tid + 256, len - 1), i2 = min(tid + 512, len - 1),
            i3 = min(tid + 768, len - 1);
  const v2d *x = reinterpret_cast<const v2d *>(v.x[0] + c0);
  const v2d a0 = x[i0], a1 = x[i1], a2 = x[i2], a3 = x[i3];
  v2d b0 = a0, b1 = a1, b2 = a2, b3 = a3;
  if constexpr (NV == 2) {
    const v2d *y = reinterpret_cast<const v2d *>(v.x[1] + c0);
    b0 = y[i0];
    b1 = y[i1];
    b2 = y[i2];
    b3 = y[i3];
  }
  __syncthreads();   // the previous chunk's shared reads are done
  v2d *o = reinterpret_cast<v2d *>(xs);
  if (tid < len) o[tid] = a0;
  if (tid + 256 < len) o[tid + 256] = a1;
  if (tid + 512 < len) o[tid + 512] = a2;
  if (tid + 768 < len) o[tid + 768] = a3;
  if constexpr (NV == 2) {
    if (tid < len) o[kMvChunk + tid] = b0;
    if (tid + 256 < len) o[kMvChunk + tid + 256] = b1;
    if (tid + 512 < len) o[kMvChunk + tid + 512] = b2;
    if (tid + 768 < len) o[kMvChunk + tid + 768] = b3;
  }
  __syncthreads();
}

template <int RPW, int NV>
__device__ __forceinline__ void matvec_body(const dz *__restrict__ Z, int64_t ld, int64_t N, const MvVecs &v,
                                            dz *xs, int blk) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t row0 = ((int64_t)blk * 4 + wave) * RPW;
  double are[NV][RPW], aim[NV][RPW];
#pragma unroll
  for (int q = 0; q < NV; ++q)
#pragma unroll
    for (int r = 0; r < RPW; ++r) are[q][r] = aim[q][r] = 0.0;
  const double *Zd = reinterpret_cast<const double *>(Z);
  for (int64_t c0 = 0; c0 < N; c0 += kMvChunk) {
    const int len = (int)min<int64_t>(kMvChunk, N - c0);
    stage_x<NV>(v, c0, len, xs);
    for (int cc = lane; cc < len; cc += 64) {
      double zr[RPW], zi[RPW];
#pragma unroll
      for (int r = 0; r < RPW; ++r) {
        const int64_t o = 2 * (min(row0 + r, N - 1) * ld + c0 + cc);
        zr[r] = __builtin_nontemporal_load(Zd + o);
        zi[r] = __builtin_nontemporal_load(Zd + o + 1);
      }
      dz xv[NV];
#pragma unroll
      for (int q = 0; q < NV; ++q) xv[q] = xs[q * kMvChunk + cc];
#pragma unroll
      for (int r = 0; r < RPW; ++r)
#pragma unroll
        for (int q = 0; q < NV; ++q) {
          are[q][r] = fma(zr[r], xv[q].re, fma(-zi[r], xv[q].im, are[q][r]));
          aim[q][r] = fma(zr[r], xv[q].im, fma(zi[r], xv[q].re, aim[q][r]));
        }
    }
  }
#pragma unroll
  for (int q = 0; q < NV; ++q)
    for (int r = 0; r < RPW; ++r) {
      const double sr = wsum(are[q][r]), si = wsum(aim[q][r]);
      const int64_t row = row0 + r;
      if (lane == 0 && row < N) {
        const dz *b = v.b[q];
        if (b) v.y[q][row] = mk(b[row].re - sr, b[row].im - si);
        else v.y[q][row] = mk(sr, si);
      }
    }
}

#define VIE_MATVEC(R)                                                                                           \
  __global__ __launch_bounds__(256) void k_matvec_r##R(const dz *__restrict__ Z, int64_t ld, int64_t N,         \
                                                       const dz *__restrict__ x, const dz *__restrict__ b,      \
                                                       dz *__restrict__ y) {                                    \
    __shared__ dz xs[kMvChunk];                                                                                 \
    const MvVecs v{{x, nullptr}, {b, nullptr}, {y, nullptr}};                                                   \
    matvec_body<R, 1>(Z, ld, N, v, xs, blockIdx.x);                                                                         \
  }                                                                                                             \
  __global__ __launch_bounds__(256) void k_matvec2_r##R(const dz *__restrict__ Z, int64_t ld, int64_t N,        \
                                                        MvVecs v) {                                             \
    __shared__ dz xs[2 * kMvChunk];                                                                             \
    matvec_body<R, 2>(Z, ld, N, v, xs, blockIdx.x);                                                                         \
  }
VIE_MATVEC(2)
VIE_MATVEC(4)
VIE_MATVEC(8)

// y = Z x (or b - Z x) for the mixed-precision operator Z = Zs + Zn: Zs the
// complex-FP32 dense far part (row-major, ld a multiple of 8), Zn the FP64
// near part in CSR.  Arithmetic and accumulation in FP64.  Same row mapping
// as k_matvec; each lane streams two adjacent FP32 entries (16 bytes) per
// row, then the wave adds its rows' near entries.
typedef float v4f __attribute__((ext_vector_type(4)));

template <int RPW, int NV>
__device__ __forceinline__ void matvec_mixed_body(const fz *__restrict__ Zs, int64_t ld, int64_t N,
                                                  const int64_t *__restrict__ rowptr,
                                                  const int32_t *__restrict__ cols, const dz *__restrict__ vals,
                                                  const MvVecs &v, dz *xs, int blk) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t row0 = ((int64_t)blk * 4 + wave) * RPW;
  double are[NV][RPW], aim[NV][RPW];
#pragma unroll
  for (int q = 0; q < NV; ++q)
#pragma unroll
    for (int r = 0; r < RPW; ++r) are[q][r] = aim[q][r] = 0.0;
  for (int64_t c0 = 0; c0 < N; c0 += kMvChunk) {
    const int len = (int)min<int64_t>(kMvChunk, N - c0);
    stage_x<NV>(v, c0, len, xs);
    for (int cc = 2 * lane; cc < len; cc += 128) {
      v4f z[RPW];
#pragma unroll
      for (int r = 0; r < RPW; ++r)
        z[r] = __builtin_nontemporal_load(reinterpret_cast<const v4f *>(Zs + min(row0 + r, N - 1) * ld + c0 + cc));
      dz x0[NV], x1[NV];
#pragma unroll
      for (int q = 0; q < NV; ++q) {
        x0[q] = xs[q * kMvChunk + cc];
        x1[q] = cc + 1 < len ? xs[q * kMvChunk + cc + 1] : mk(0, 0);
      }
#pragma unroll
      for (int r = 0; r < RPW; ++r)
#pragma unroll
        for (int q = 0; q < NV; ++q) {
          are[q][r] = fma((double)z[r][0], x0[q].re, fma(-(double)z[r][1], x0[q].im, are[q][r]));
          aim[q][r] = fma((double)z[r][0], x0[q].im, fma((double)z[r][1], x0[q].re, aim[q][r]));
          are[q][r] = fma((double)z[r][2], x1[q].re, fma(-(double)z[r][3], x1[q].im, are[q][r]));
          aim[q][r] = fma((double)z[r][2], x1[q].im, fma((double)z[r][3], x1[q].re, aim[q][r]));
        }
    }
  }
#pragma unroll
  for (int r = 0; r < RPW; ++r) {
    const int64_t row = row0 + r;
    if (row < N)
      for (int64_t e = rowptr[row] + lane; e < rowptr[row + 1]; e += 64) {
        const dz nv = vals[e];
        const int c = cols[e];
#pragma unroll
        for (int q = 0; q < NV; ++q) {
          const dz xv = v.x[q][c];
          are[q][r] = fma(nv.re, xv.re, fma(-nv.im, xv.im, are[q][r]));
          aim[q][r] = fma(nv.re, xv.im, fma(nv.im, xv.re, aim[q][r]));
        }
      }
  }
#pragma unroll
  for (int q = 0; q < NV; ++q)
    for (int r = 0; r < RPW; ++r) {
      const double sr = wsum(are[q][r]), si = wsum(aim[q][r]);
      const int64_t row = row0 + r;
      if (lane == 0 && row < N) {
        const dz *b = v.b[q];
        if (b) v.y[q][row] = mk(b[row].re - sr, b[row].im - si);
        else v.y[q][row] = mk(sr, si);
      }
    }
}

#define VIE_MATVEC_MIXED(R)                                                                                     \
  __global__ __launch_bounds__(256) void k_matvec_mixed_r##R(                                                   \
      const fz *__restrict__ Zs, int64_t ld, int64_t N, const int64_t *__restrict__ rowptr,                     \
      const int32_t *__restrict__ cols, const dz *__restrict__ vals, const dz *__restrict__ x,                  \
      const dz *__restrict__ b, dz *__restrict__ y) {                                                           \
    __shared__ dz xs[kMvChunk];                                                                                 \
    const MvVecs v{{x, nullptr}, {b, nullptr}, {y, nullptr}};                                                   \
    matvec_mixed_body<R, 1>(Zs, ld, N, rowptr, cols, vals, v, xs, blockIdx.x);                                              \
  }                                                                                                             \
  __global__ __launch_bounds__(256) void k_matvec2_mixed_r##R(                                                  \
      const fz *__restrict__ Zs, int64_t ld, int64_t N, const int64_t *__restrict__ rowptr,                     \
      const int32_t *__restrict__ cols, const dz *__restrict__ vals, MvVecs v) {                                \
    __shared__ dz xs[2 * kMvChunk];                                                                             \
    matvec_mixed_body<R, 2>(Zs, ld, N, rowptr, cols, vals, v, xs, blockIdx.x);                                              \
  }
VIE_MATVEC_MIXED(2)
VIE_MATVEC_MIXED(4)
VIE_MATVEC_MIXED(8)

// y[k] = sum_{i<nv} V_i[k] c[i]
__global__ __launch_bounds__(256) void k_combine(const dz *__restrict__ V, int64_t ldv, int nv,
                                                 const dz *__restrict__ c, dz *__restrict__ y, int64_t N) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= N) return;
  dz s = mk(0, 0);
  // eight basis entries in flight at a time; the sum runs in i order
  for (int i0 = 0; i0 < nv; i0 += 8) {
    double vr[8], vi[8];
#pragma unroll
    for (int g = 0; g < 8; ++g) {
      const dz v = V[(int64_t)min(i0 + g, nv - 1) * ldv + k];
      vr[g] = v.re;
      vi[g] = v.im;
    }
#pragma unroll
    for (int g = 0; g < 8; ++g)
      if (i0 + g < nv) s = s + mk(vr[g], vi[g]) * c[i0 + g];
  }
  y[k] = s;
}

// partial squared norms per block
__global__ __launch_bounds__(256) void k_norm2(const dz *__restrict__ w, int64_t N, double *__restrict__ part) {
  __shared__ double red[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t chunk = (N + gridDim.x - 1) / gridDim.x;
  const int64_t lo = blockIdx.x * chunk, hi = min<int64_t>(N, lo + chunk);
  double s = 0;
  for (int64_t k = lo + tid; k < hi; k += 256) s = fma(w[k].re, w[k].re, fma(w[k].im, w[k].im, s));
  s = wsum(s);
  if (lane == 0) red[wave] = s;
  __syncthreads();
  if (tid == 0) part[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

// out = sqrt(sum part)
__global__ void k_norm_reduce(const double *__restrict__ part, int nblk, double *__restrict__ out) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  double s = 0;
  for (int b0 = 0; b0 < nblk; b0 += 16) {   // sixteen loads in flight, summed in order
    double p[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) p[u] = part[min(b0 + u, nblk - 1)];
#pragma unroll
    for (int u = 0; u < 16; ++u)
      if (b0 + u < nblk) s += p[u];
  }
  *out = sqrt(s);
}

// v = vin = w / *nrm (the first basis vector, which the first step takes)
__global__ void k_scale(const dz *__restrict__ w, const double *__restrict__ nrm, dz *__restrict__ v,
                        dz *__restrict__ vin, int64_t N) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= N) return;
  const dz x = (1.0 / *nrm) * w[k];
  v[k] = x;
  vin[k] = x;
}

__global__ void k_axpy(dz *__restrict__ x, const dz *__restrict__ u, int64_t N) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < N) x[k] = x[k] + u[k];
}

// 1 / Z_mm (one thread per row).  Z_mm sums the dense entry (FP64, or the
// FP32 far part) and the row's CSR slot for column m when there is a near
// part; a zero diagonal (no physical operator has one) leaves the row unscaled.
__global__ void k_jacobi_diag(int64_t N, ZOut Z, dz *__restrict__ dinv) {
  const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= N) return;
  dz d = mk(0.0, 0.0);
  if (Z.Z) d = Z.Z[m * Z.ld + m];
  if (Z.Zs) d = mk((double)Z.Zs[m * Z.ld + m].re, (double)Z.Zs[m * Z.ld + m].im);
  if (Z.rowptr) {
    int64_t lo = Z.rowptr[m], hi = Z.rowptr[m + 1];
    while (lo < hi) {
      const int64_t mid = (lo + hi) >> 1;
      if (Z.cols[mid] < m) lo = mid + 1;
      else hi = mid;
    }
    if (lo < Z.rowptr[m + 1] && Z.cols[lo] == m) d = d + Z.vals[lo];
  }
  const double den = d.re * d.re + d.im * d.im;
  dinv[m] = den > 0.0 ? mk(d.re / den, -d.im / den) : mk(1.0, 0.0);
}

__global__ void k_jacobi_apply(int64_t N, const dz *__restrict__ dinv, const dz *__restrict__ v, dz *__restrict__ z) {
  const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (m < N) z[m] = dinv[m] * v[m];
}

__global__ void k_fill_const(dz *__restrict__ x, int64_t N, double re, double im) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < N) x[k] = mk(re, im);
}

__global__ void k_copy(dz *__restrict__ d, const dz *__restrict__ s, int64_t N) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < N) d[k] = s[k];
}

// ------------------------------------------------------------ Arnoldi step
// After the preconditioner and the product, a step is five launches for all
// its processes together (both polarisations of a pair, every cell of a
// batch): partial inner products; their reduction and the update of w, twice
// (CGS2), the second also with partial squared norms; then V_{j+1} and the
// Givens update.  Each is a few microseconds of latency, not of bandwidth, so
// reductions are finished by the blocks that use them (each reads all the
// partials) rather than in launches of their own: one reduction or one scalar
// kernel per process took 11 launches and 80 us per process and step at
// N = 6,272 (five and 35 us now, for both).  The kernels read the column index j
// from device memory, so the step issues the same launches for every j and can
// be captured once in a HIP graph and replayed.  Nothing reads *jd in the last
// launch, which advances it (j is handed to it in jd[1]).

// partial inner products with V_0 .. V_j: block (bx, by) sums chunk bx of the
// nd chunks of N for basis vectors 8 by .. 8 by + 7 (their loads in flight
// together, one barrier for the eight sums; blocks past V_j return at once)
template <class K>
__device__ __forceinline__ void kry_dots(const K &k, int bx, int by) {
  constexpr int G = 8;
  __shared__ dz red[G][4];
  const int nv = *k.jd + 1;
  const int i0 = by * G;
  if (i0 >= nv) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t N = k.N, ldv = k.ldv;
  const int64_t chunk = (N + k.nd - 1) / k.nd;
  const int64_t lo = bx * chunk, hi = min<int64_t>(N, lo + chunk);
  double sr[G], si[G];
#pragma unroll
  for (int g = 0; g < G; ++g) sr[g] = si[g] = 0.0;
  for (int64_t e = lo + tid; e < hi; e += 256) {
    const dz ww = k.w[e];
    double vr[G], vi[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const dz v = k.V[(int64_t)min(i0 + g, nv - 1) * ldv + e];
      vr[g] = v.re;
      vi[g] = v.im;
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      sr[g] = fma(vr[g], ww.re, fma(vi[g], ww.im, sr[g]));
      si[g] = fma(vr[g], ww.im, fma(-vi[g], ww.re, si[g]));
    }
  }
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const double a = wsum(sr[g]), b = wsum(si[g]);
    if (lane == 0) red[g][wave] = mk(a, b);
  }
  __syncthreads();
  if (tid < G && i0 + tid < nv)
    k.dpart[(int64_t)bx * nv + i0 + tid] = red[tid][0] + red[tid][1] + red[tid][2] + red[tid][3];
}

// s_i = sum over the nd partials; w -= sum_{i<=j} V_i s_i over the rows of
// block b (of nupd, strided); block 0 stores H[i][j] = s_i (pass 0) or += s_i
// (pass 1).  64 basis vectors at a time: four waves sum a quarter of the
// partials each (16 loads in flight), then every thread updates its rows.
// Pass 1: also the block's sum of |w|^2 into npart[b], and j for the last launch.
template <class K>
__device__ __forceinline__ void kry_update(const K &k, int b, int pass) {
  constexpr int T = 64;
  __shared__ dz q[4][T], c[T];
  __shared__ double red[4];
  const int j = *k.jd, nv = j + 1;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t N = k.N, first = (int64_t)b * 256 + tid, stride = (int64_t)k.nupd * 256;
  if (b == 0 && tid == 0) k.jd[1] = j;
  double nrm = 0.0;
  for (int t0 = 0; t0 < nv; t0 += T) {
    const int nt = min(T, nv - t0);
    {
      const int i = t0 + min(lane, nt - 1);
      dz s = mk(0, 0);
      for (int b0 = wave; b0 < k.nd; b0 += 64) {
        double pr[16], pi[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
          const dz p = k.dpart[(int64_t)min(b0 + 4 * u, k.nd - 1) * nv + i];
          pr[u] = p.re;
          pi[u] = p.im;
        }
#pragma unroll
        for (int u = 0; u < 16; ++u)
          if (b0 + 4 * u < k.nd) s = s + mk(pr[u], pi[u]);
      }
      q[wave][lane] = s;
    }
    __syncthreads();
    if (tid < nt) {
      const dz s = (q[0][tid] + q[1][tid]) + (q[2][tid] + q[3][tid]);
      c[tid] = s;
      if (b == 0) {
        dz *h = k.H + (int64_t)j * k.ldh + t0 + tid;
        *h = pass ? *h + s : s;
      }
    }
    __syncthreads();
    const bool last = t0 + T >= nv;
    for (int64_t e = first; e < N; e += stride) {
      dz s = k.w[e];
      // eight basis entries in flight at a time; the updates run in i order
      for (int g0 = 0; g0 < nt; g0 += 8) {
        double vr[8], vi[8];
#pragma unroll
        for (int g = 0; g < 8; ++g) {
          const dz v = k.V[(int64_t)(t0 + min(g0 + g, nt - 1)) * k.ldv + e];
          vr[g] = v.re;
          vi[g] = v.im;
        }
#pragma unroll
        for (int g = 0; g < 8; ++g)
          if (g0 + g < nt) s = s - mk(vr[g], vi[g]) * c[g0 + g];
      }
      k.w[e] = s;
      if (last) nrm = fma(s.re, s.re, fma(s.im, s.im, nrm));
    }
    __syncthreads();   // c and q may be reused
  }
  if (!pass) return;
  nrm = wsum(nrm);
  if (lane == 0) red[wave] = nrm;
  __syncthreads();
  if (tid == 0) k.npart[b] = (red[0] + red[1]) + (red[2] + red[3]);
}

__global__ void k_jset(int *__restrict__ jd, int v) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *jd = v;
}

// GMRES state on the device: H (ldh x m, column j holds h_{0..j+1, j}),
// Givens cosines (real) and sines (complex), g (m+1).
// Arnoldi column j: h[0..j] from CGS2, hn = ||w||.  Apply the previous
// rotations to column j, form the new one, update g, write |g[j+1]| (to *hist
// and, if given, *res).  Called by a whole block of 256 threads: the column and
// the rotations go through LDS, 128 at a time, and one thread applies them (a
// chain over j; from global memory it was 8.8 us at j = 30).
__device__ __forceinline__ void givens_step(dz *__restrict__ H, int ldh, int j, double hnv, double *__restrict__ cs,
                                            dz *__restrict__ sn, dz *__restrict__ g, double *__restrict__ hist,
                                            double *__restrict__ res) {
  constexpr int T = 128;
  __shared__ dz hh[T + 1], ss[T];
  __shared__ double cc[T];
  dz *h = H + (int64_t)j * ldh;
  const int tid = threadIdx.x;
  dz a = mk(0, 0), b = mk(0, 0);   // thread 0: the entry carried to the next rotation
  for (int i0 = 0; i0 < j; i0 += T) {
    const int nt = min(T, j - i0);
    if (tid < nt) {
      ss[tid] = sn[i0 + tid];
      cc[tid] = cs[i0 + tid];
    }
    if (tid <= nt) hh[tid] = h[i0 + tid];
    __syncthreads();
    if (tid == 0) {
      a = i0 == 0 ? hh[0] : a;
      for (int i = 0; i < nt; ++i) {
        // [c  s; -conj(s) c] acting on (h_i, h_{i+1})
        b = hh[i + 1];
        hh[i] = cc[i] * a + ss[i] * b;
        a = cc[i] * b - conjz(ss[i]) * a;
      }
    }
    __syncthreads();
    if (tid < nt) h[i0 + tid] = hh[tid];
    __syncthreads();
  }
  if (tid != 0) return;
  if (j == 0) a = h[0];
  b = mk(hnv, 0.0);
  const double na = sqrt(a.re * a.re + a.im * a.im), nb = hnv;
  double c;
  dz s;
  if (na == 0.0) {
    c = 0.0;
    s = mk(1.0, 0.0);
    h[j] = b;
  } else {
    const double t = sqrt(na * na + nb * nb);
    c = na / t;
    const dz al = mk(a.re / na, a.im / na);       // a / |a|
    s = (1.0 / t) * (al * conjz(b));              // alpha conj(b) / t
    h[j] = al * mk(t, 0.0);
  }
  h[j + 1] = mk(0.0, 0.0);
  cs[j] = c;
  sn[j] = s;
  const dz gj = g[j];
  g[j] = c * gj;
  const dz gn = mk(0, 0) - conjz(s) * gj;
  g[j + 1] = gn;
  const double r = sqrt(gn.re * gn.re + gn.im * gn.im);
  *hist = r;
  if (res) *res = r;
}

// h_{j+1,j} = ||w|| from the nupd partials; V_{j+1} = w / h_{j+1,j}, also into
// vin, over the rows of block b; block 0 then takes the Givens step on column
// j (|g_{j+1}| into rhist[j] and *res) and advances *jd.
template <class K>
__device__ __forceinline__ void kry_finish(const K &k, int b, double *res) {
  __shared__ double red[4];
  const int j = k.jd[1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double s = 0.0;
  for (int i = tid; i < k.nupd; i += 256) s += k.npart[i];
  s = wsum(s);
  if (lane == 0) red[wave] = s;
  __syncthreads();
  const double hn = sqrt((red[0] + red[1]) + (red[2] + red[3])), sc = 1.0 / hn;
  dz *v = k.V + (int64_t)(j + 1) * k.ldv;
  for (int64_t e = (int64_t)b * 256 + tid; e < k.N; e += (int64_t)k.nupd * 256) {
    const dz x = sc * k.w[e];
    v[e] = x;
    k.vin[e] = x;
  }
  if (b > 0) return;
  givens_step(k.H, k.ldh, j, hn, k.cs, k.sn, k.g, k.rhist + j, res);
  if (tid == 0) k.jd[0] = j + 1;
}

__global__ __launch_bounds__(256) void k_kry_dots(KryPair P) { kry_dots(P.p[blockIdx.z], blockIdx.x, blockIdx.y); }
__global__ __launch_bounds__(256) void k_kry_update(KryPair P, int pass) { kry_update(P.p[blockIdx.y], blockIdx.x, pass); }
__global__ __launch_bounds__(256) void k_kry_finish(KryPair P) { kry_finish(P.p[blockIdx.y], blockIdx.x, nullptr); }

// y = R^{-1} g for the leading k x k upper triangle of H (single thread).
__global__ void k_backsolve(const dz *__restrict__ H, int ldh, int k, const dz *__restrict__ g, dz *__restrict__ y) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  for (int i = k - 1; i >= 0; --i) {
    dz s = g[i];
    for (int l = i + 1; l < k; ++l) s = s - H[(int64_t)l * ldh + i] * y[l];
    const dz d = H[(int64_t)i * ldh + i];
    const double den = d.re * d.re + d.im * d.im;
    y[i] = mk((s.re * d.re + s.im * d.im) / den, (s.im * d.re - s.re * d.im) / den);
  }
}

// g = (beta, 0, ..., 0)
__global__ void k_ginit(dz *__restrict__ g, int m1, const double *__restrict__ beta) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < m1) g[i] = i == 0 ? mk(*beta, 0.0) : mk(0.0, 0.0);
}

// ------------------------------------------------------------ fused batch
// The Arnoldi step of many cells at once (one GMRES process per cell): each
// kernel's grid is the concatenation of the cells' grids (pre[c] .. pre[c+1]
// are cell c's blocks), and a cell whose flag act[c] is 0 skips the step.
// Per cell the arithmetic is that of the single-cell kernels.

__device__ __forceinline__ int cell_of(const int *__restrict__ pre, int nc, int b) {
  int lo = 0, hi = nc - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (pre[mid] <= b) lo = mid;
    else hi = mid - 1;
  }
  return __builtin_amdgcn_readfirstlane(lo);
}

#define VIE_CELL_BEGIN                                \
  const int c_ = cell_of(pre, nc, (int)blockIdx.x);   \
  if (!act[c_]) return;                               \
  const KryCell &K = cells[c_];                       \
  const int lb = (int)blockIdx.x - pre[c_];

// rhs of the triangular solves: tmp[off + i] = vin[off + perm[off + i]] per domain
__global__ void k_b_permute(const KryCell *__restrict__ cells, const int *__restrict__ pre, int nc,
                            const int *__restrict__ act) {
  VIE_CELL_BEGIN
  const int64_t k = (int64_t)lb * blockDim.x + threadIdx.x;
  if (k >= K.N) return;
  int64_t off = 0;
  for (int d = 1; d < K.ndom; ++d)
    if (k >= K.dstart[d]) off = K.dstart[d];
  K.tmp[k] = K.vin[off + K.perm[k]];
}

// w = Z z (the operator of the cell's precision); z = vin when unpreconditioned
__global__ __launch_bounds__(256) void k_b_matvec(const KryCell *__restrict__ cells, const int *__restrict__ pre, int nc,
                                                  const int *__restrict__ act) {
  __shared__ dz xs[kMvChunk];
  VIE_CELL_BEGIN
  const MvVecs v{{K.precond ? K.vin : K.z, nullptr}, {nullptr, nullptr}, {K.w, nullptr}};
  // rows per wave: the cell's autotuned shape
  if (K.Z) {
    if (K.rpw == 2) matvec_body<2, 1>(K.Z, K.ld, K.N, v, xs, lb);
    else if (K.rpw == 8) matvec_body<8, 1>(K.Z, K.ld, K.N, v, xs, lb);
    else matvec_body<4, 1>(K.Z, K.ld, K.N, v, xs, lb);
  } else {
    if (K.rpw == 2) matvec_mixed_body<2, 1>(K.Zs, K.ld, K.N, K.rowptr, K.cols, K.vals, v, xs, lb);
    else if (K.rpw == 8) matvec_mixed_body<8, 1>(K.Zs, K.ld, K.N, K.rowptr, K.cols, K.vals, v, xs, lb);
    else matvec_mixed_body<4, 1>(K.Zs, K.ld, K.N, K.rowptr, K.cols, K.vals, v, xs, lb);
  }
}

// the five launches of the step: local block lb of the cell
__global__ __launch_bounds__(256) void k_b_dots(const KryCell *__restrict__ cells, const int *__restrict__ pre, int nc,
                                                const int *__restrict__ act) {
  VIE_CELL_BEGIN
  kry_dots(K, lb % K.nd, lb / K.nd);
}
__global__ __launch_bounds__(256) void k_b_update(const KryCell *__restrict__ cells, const int *__restrict__ pre, int nc,
                                                  const int *__restrict__ act, int pass) {
  VIE_CELL_BEGIN
  kry_update(K, lb, pass);
}
// (the step's residual estimate |g_{j+1}| into res[c])
__global__ __launch_bounds__(256) void k_b_finish(const KryCell *__restrict__ cells, const int *__restrict__ pre, int nc,
                                                  const int *__restrict__ act, double *__restrict__ res) {
  VIE_CELL_BEGIN
  kry_finish(K, lb, res + c_);
}
#undef VIE_CELL_BEGIN

}  // namespace vie
