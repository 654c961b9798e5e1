// Application of the block-diagonal preconditioner of Sec. 2.3 (Eq. 6)
// inside GMRES: z = A_dd^{-1} v for every material domain d, from the LU
// factors of k_lu.hip, by a permutation and blocked forward (L, unit lower)
// and backward (U) substitutions over 512-row diagonal blocks; the inverses
// of the diagonal blocks and the coupling blocks the substitutions use are
// formed once per factorisation.
#include <hip/hip_cooperative_groups.h>
#include <hip/hip_runtime.h>

#include "kernels.h"

namespace vie {

// ------------------------------------------------------------ apply
// z[i] = v[perm[i]] for one block (offset `off` in the global vectors)
__global__ void k_permute(int n, int64_t off, const int32_t *__restrict__ perm, const dz *__restrict__ v,
                          dz *__restrict__ z) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) z[off + i] = v[off + perm[i]];
}

// Inverses of the kTrsvNB x kTrsvNB diagonal blocks of L (unit lower) and U
// (upper), computed once per factorisation: block b of INV, at b nb^2,
// holds inv(T_bb) row-major with its own size m (nb but for a domain's last
// block) as leading dimension, T_bb the diagonal block at row b*nb.
//
// A thread block forms 16 columns of one inverse by substitution over 16-row
// strips, the columns held in LDS in FP64 (128 KB: one thread block per CU).
// Strip r is rhs - sum_l T[r, l] X[l] over the strips l solved so far, on the
// FP64 matrix cores: the four waves take the strips l in turn, their partial
// sums meet in LDS, and wave 0 finishes the strip with its 16 x 16 diagonal
// block, four rows and one column per lane.  U is taken with rows and columns
// reversed, where it is a lower triangle too.  What bounds it is the chain of
// up to 32 strips: a substitution with one lane quad per column, a chain of
// 512 rows, took 1.9-4.1 ms per launch and two launches per domain.  The L and
// U inverses of up to kLuMaxDom domains share one launch: 0.20 ms for N = 416
// (3.98 before), 0.98 ms for N = 15,840 in three domains, FP64 (24.4 before).
typedef double v4d __attribute__((ext_vector_type(4)));

template <typename C>
__device__ __forceinline__ void diag_inv_body(const TrsvPrep &st) {
  constexpr int S = 16;
  __shared__ dz X[kTrsvNB][S];
  __shared__ dz P[4][S][S];
  __shared__ dz Td[S][S + 1];
  int dd = 0;
  while (dd + 1 < st.ndom && (int)blockIdx.x >= st.d[dd + 1].first_block) ++dd;
  const TrsvPrepDom &D = st.d[dd];
  const int b = blockIdx.x - D.first_block, n = D.n;
  const bool lower = blockIdx.z == 0;
  const int b0 = b * kTrsvNB, m = min(kTrsvNB, n - b0), c = blockIdx.y;
  if (c * S >= m) return;
  const int64_t ld = D.ld;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, col = lane & 15, g = lane >> 4;
  // element (i, l) of the (reversed, for U) lower triangle: base + dir (i ld + l)
  const int64_t dir = lower ? 1 : -1;
  const C *__restrict__ T = (const C *)D.F + (int64_t)b0 * ld + b0 + (lower ? 0 : (int64_t)(m - 1) * (ld + 1));
  const int ns = (m + S - 1) / S;
  for (int r = c; r < ns; ++r) {
    // the strip's diagonal block, one entry per thread (identity past the block's size)
    {
      const int i = r * S + tid / S, l = r * S + tid % S;
      const dz t = to_dz(T[dir * (min(i, m - 1) * ld + min(l, m - 1))]);
      Td[tid / S][tid % S] = i < m && l < m ? t : mk(i == l ? 1.0 : 0.0, 0.0);
    }
    v4d cre = {0, 0, 0, 0}, cim = {0, 0, 0, 0};
    const int row = min(r * S + col, m - 1);   // (rows past the block repeat its last; their strip rows are not stored)
    for (int l = c + wave; l < r; l += 4) {
      // the k index of MFMA step s is 4 g + s in both operands: a lane reads four neighbours of its row
      const C *Tl = T + dir * (row * ld + l * S + 4 * g);
      C a[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) a[s] = Tl[dir * s];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const dz av = to_dz(a[s]), x = X[l * S + 4 * g + s][col];
        cre = __builtin_amdgcn_mfma_f64_16x16x4f64(av.re, x.re, cre, 0, 0, 0);
        cim = __builtin_amdgcn_mfma_f64_16x16x4f64(av.re, x.im, cim, 0, 0, 0);
        cre = __builtin_amdgcn_mfma_f64_16x16x4f64(-av.im, x.im, cre, 0, 0, 0);
        cim = __builtin_amdgcn_mfma_f64_16x16x4f64(av.im, x.re, cim, 0, 0, 0);
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) P[wave][4 * q + g][col] = mk(cre[q], cim[q]);
    __syncthreads();
    if (wave == 0) {
      dz v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = 4 * g + q;
        const dz s = (P[0][i][col] + P[1][i][col]) + (P[2][i][col] + P[3][i][col]);
        v[q] = mk((r == c && i == col ? 1.0 : 0.0) - s.re, -s.im);
      }
#pragma unroll
      for (int k = 0; k < S; ++k) {
        dz xk = v[k & 3];
        if (!lower) {   // U: divide by the diagonal entry
          const dz d = Td[k][k];
          const double den = d.re * d.re + d.im * d.im;
          xk = xk * mk(d.re / den, -d.im / den);
        }
        if (g == k >> 2) v[k & 3] = xk;
        const int src = (k >> 2) * S + col;
        xk = mk(__shfl(xk.re, src), __shfl(xk.im, src));
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (4 * g + q > k) cmac(v[q], mk(-Td[4 * g + q][k].re, -Td[4 * g + q][k].im), xk);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) X[r * S + 4 * g + q][col] = v[q];
    }
    __syncthreads();
  }
  // the inverse of block b, m x m row-major: its columns c S .. (zero above the first strip)
  C *__restrict__ inv_b = (C *)(lower ? D.INVL : D.INVU) + (int64_t)b * kTrsvNB * kTrsvNB;
  const int j = c * S + tid % S;
  if (j >= m) return;
  for (int i = tid / S; i < m; i += S) {
    const dz v = i >= c * S ? X[i][tid % S] : mk(0, 0);
    inv_b[lower ? (int64_t)i * m + j : (int64_t)(m - 1 - i) * m + (m - 1 - j)] = cx<C>::of(v);
  }
}

__global__ __launch_bounds__(256) void k_diag_inv_z(TrsvPrep st) { diag_inv_body<dz>(st); }
__global__ __launch_bounds__(256) void k_diag_inv_c(TrsvPrep st) { diag_inv_body<fz>(st); }

// Coupling blocks of a domain's sweeps: for the matrix blocks b that follow
// another in the sweep's order (b >= 1 for L, b <= nbk - 2 for U), with p =
// b - 1 (L) or b + 1 (U), G_b = T[b, p] inv(T_pp), a kTrsvNB x kTrsvNB
// product in FP64 (rounded to the factor type), written to slot b - 1 (L) or
// b (U) of nb^2 entries, leading dimension nb.  A thread block forms a 64 x 64
// tile on the FP64 matrix cores, 2 x 2 waves of 2 x 2 instruction tiles, through
// 16-deep slices of both operands in shared memory, the next slice's loads in
// flight; entries past the blocks' sizes are zero, and slices in which the
// triangle inv(T_pp) is zero are left out (half of them).  All domains' L and U
// blocks share a launch.  The matrix cores' FP64 rate bounds it: N = 15,840, FP64, 0.72
// ms, six FP32 cells of up to 5,500 1.19 ms (1.80 and 2.41 with FMAs, 4 x 4
// entries per thread, over all slices).
template <typename C>
__device__ __forceinline__ void coupling_body(const TrsvPrep &st) {
  constexpr int nb = kTrsvNB, TS = 64, KS = 16, kPer = TS * KS / 256;
  __shared__ double Ar[TS][KS + 1], Ai[TS][KS + 1], Br[KS][TS + 1], Bi[KS][TS + 1];
  int dd = 0;
  while (dd + 1 < st.ndom && (int)blockIdx.x >= st.d[dd + 1].first_block) ++dd;
  const TrsvPrepDom &D = st.d[dd];
  const bool lower = blockIdx.z == 0;
  const C *__restrict__ F = (const C *)D.F, *__restrict__ INV = (const C *)(lower ? D.INVL : D.INVU);
  C *__restrict__ G = (C *)(lower ? D.GL : D.GU);
  const int64_t ld = D.ld;
  const int n = D.n, pb = blockIdx.x - D.first_block;
  const int b = lower ? pb + 1 : pb;
  const int p = lower ? b - 1 : b + 1;
  const int b0 = b * nb, p0 = p * nb;
  const int mr = min(nb, n - b0), mc = min(nb, n - p0);
  const int r0 = blockIdx.y / (nb / TS) * TS, c0 = blockIdx.y % (nb / TS) * TS;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32, li = lane & 15, lg = lane >> 4;
  const C *__restrict__ Ip = INV + (int64_t)p * nb * nb;   // mc x mc, leading dimension mc
  v4d cre[2][2], cim[2][2];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int v = 0; v < 2; ++v) cre[u][v] = cim[u][v] = v4d{0, 0, 0, 0};
  // inv(T_pp) is zero above (L) or below (U) its diagonal: rows k of column tile c0
  const int kbeg = lower ? c0 : 0, kend = r0 < mr && c0 < mc ? min(mc, lower ? nb : c0 + TS) : 0;
  C va[kPer], vb[kPer];
  const auto fetch = [&](int k0) {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int e = tid + 256 * u;
      va[u] = F[(int64_t)(b0 + min(r0 + e / KS, mr - 1)) * ld + p0 + min(k0 + e % KS, mc - 1)];
      vb[u] = Ip[(int64_t)min(k0 + e / TS, mc - 1) * mc + min(c0 + e % TS, mc - 1)];
    }
  };
  if (kbeg < kend) fetch(kbeg);
  for (int k0 = kbeg; k0 < kend; k0 += KS) {
    __syncthreads();   // the previous slice's shared reads are done
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int e = tid + 256 * u;
      const bool ka = r0 + e / KS < mr && k0 + e % KS < mc, kb = k0 + e / TS < mc && c0 + e % TS < mc;
      const dz a = to_dz(va[u]), v = to_dz(vb[u]);
      Ar[e / KS][e % KS] = ka ? a.re : 0.0;
      Ai[e / KS][e % KS] = ka ? a.im : 0.0;
      Br[e / TS][e % TS] = kb ? v.re : 0.0;
      Bi[e / TS][e % TS] = kb ? v.im : 0.0;
    }
    __syncthreads();
    fetch(min(k0 + KS, mc - 1));   // the next slice (clamped; unused past the end)
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kk = 0; kk < KS; kk += 4) {
      double are[2], aim[2], bre[2], bim[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        are[u] = Ar[wr + 16 * u + li][kk + lg];
        aim[u] = Ai[wr + 16 * u + li][kk + lg];
        bre[u] = Br[kk + lg][wc + 16 * u + li];
        bim[u] = Bi[kk + lg][wc + 16 * u + li];
      }
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v) {
          cre[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(are[u], bre[v], cre[u][v], 0, 0, 0);
          cim[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(are[u], bim[v], cim[u][v], 0, 0, 0);
        }
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v) {
          cre[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(-aim[u], bim[v], cre[u][v], 0, 0, 0);
          cim[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(aim[u], bre[v], cim[u][v], 0, 0, 0);
        }
    }
  }
  C *__restrict__ Gb = G + (int64_t)(lower ? b - 1 : b) * nb * nb;   // slots of the sweep's nbk - 1 blocks
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        Gb[(int64_t)(r0 + wr + 16 * u + 4 * q + lg) * nb + c0 + wc + 16 * v + li] = cx<C>::of(mk(cre[u][v][q], cim[u][v][q]));
}
__global__ __launch_bounds__(256) void k_trsv_coupling_z(TrsvPrep st) { coupling_body<dz>(st); }
__global__ __launch_bounds__(256) void k_trsv_coupling_c(TrsvPrep st) { coupling_body<fz>(st); }

__device__ __forceinline__ dz wave_sum(dz v) {
  for (int o = 32; o > 0; o >>= 1) {
    v.re += __shfl_xor(v.re, o);
    v.im += __shfl_xor(v.im, o);
  }
  return v;
}

// One step of the blocked triangular solves (L forward or U backward) of
// every material domain at once, with nb = kTrsvNB diagonal blocks.  Blocks
// are numbered in the order of the sweep; step j of domain d reduces block j.
// Write r_k = rhs_k - sum over i < k of T[k, i] z_i, so that z_k =
// inv(T_kk) r_k, and precompute per block the coupling G_k = T[k, k-1]
// inv(T_{k-1,k-1}), for which T[k, k-1] z_{k-1} = G_k r_{k-1}.  On entry
//   - z_{j-2}, block [cb0, cb0+cm), is in sol (cm = 0 if j < 2);
//   - r_{j-1} of block [pb0, pb0+pm) is in rin (pm = 0 if j < 1);
//   - for every row of block j, the sum of T[i, k] z_k over the blocks k < j-2
//     is in bsum_in as nci chunk sums (nci = 0 if j < 3).
// The launch has three kinds of work items, numbered in this order:
//   (1) reduction items, 16 rows of block j each:
//       r_j = rhs_j - (its chunk sums) - T[j, j-2] z_{j-2} - G_j r_{j-1},
//       written to rout (the next step's rin);
//   (2) solution items, 16 rows of block j-1 each: z_{j-1} = inv(T_{j-1,j-1})
//       r_{j-1}, written to sol;
//   (3) chunk-sum items: for the rows of block j+1 (if any), the sums of
//       T[i, k] z_k over the blocks k <= j-2 (solutions in sol), columns
//       [bc0, bc0+bk) in chunks of kTrsvSumCols, into bsum_out.
// Only (1) is on the step-to-step chain: one stage of loads, one barrier and
// one dot product per row.  The update reads of (3) run along factor rows,
// so each launch streams whole row segments rather than a strip of one block
// column.  An entry with nm = 0 (the end of a sweep) has only solution items.
// No thread block waits on another; the right-hand sides are only read.
constexpr int kTrsvGroups = kTrsvGroupsH;
constexpr int kTrsvCol = kTrsvNB / 64;   // column chunks of 64 per row

// Loads in these kernels are unconditional, from addresses clamped into the
// domain's arrays, with out-of-range values zeroed afterwards: a load under a
// branch is waited for inside the branch, which would serialise the loads.
__device__ __forceinline__ int clampi(int v, int hi) { return max(0, min(v, hi)); }

// A block-length vector (m entries at src_q, zero past m) of each of NV
// vectors into shared memory.  All threads load (the same addresses
// 1024 / kTrsvNB times over) so that no branch waits for the load before
// the loads that follow are issued; threads below kTrsvNB store.
template <int NV>
struct TrsvVec {
  dz v[NV];
  template <class Src>
  __device__ __forceinline__ void fetch(Src src, int m) {
    const int t = threadIdx.x & (kTrsvNB - 1);
#pragma unroll
    for (int q = 0; q < NV; ++q) v[q] = src(q)[clampi(t, m - 1)];
  }
  __device__ __forceinline__ void store(dz *dst, int m) const {   // dst[q * kTrsvNB + t]
    const int t = threadIdx.x;
    if (t >= kTrsvNB) return;
#pragma unroll
    for (int q = 0; q < NV; ++q) dst[q * kTrsvNB + t] = t < m ? v[q] : mk(0, 0);
  }
};

// Shared memory of a step's thread block: reduction and solution items use
// two block-length vectors per right-hand side, chunk-sum items the chunk's
// solutions; one array serves all.
template <int NV, int KC>
struct TrsvLds {
  static constexpr int kChain = 2 * NV * kTrsvNB;
  static constexpr int kChunk = NV * KC;
  static constexpr int kSize = kChain > kChunk ? kChain : kChunk;
};

// KC columns per chunk-sum item (the autotuner picks 1024 or 2048 per
// context; the sums are the same).  NV right-hand sides (1 or 2) share each
// read of the factors; vector q's sums run in the same order for any NV.
template <typename C, int KC, int NV, typename ST = TrsvStep>
__device__ __forceinline__ void trsv_step_body(const ST &st, int vb) {
  static_assert(KC % 1024 == 0, "chunk staging: whole passes of 1024 threads");
  __shared__ dz sm[TrsvLds<NV, KC>::kSize];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // the item's kind and domain: the last entry whose first item of that kind is <= vb
  const int kind = vb < st.chain_blocks ? 0 : (vb < st.z_end ? 1 : 2);
  int d = 0;
  for (int lo = 0, hi = st.ndom - 1; lo <= hi;) {
    const int mid = (lo + hi) >> 1;
    const TrsvDom &M = st.d[mid];
    if ((kind == 0 ? M.first_block : kind == 1 ? M.first_z : M.first_bulk) <= vb) {
      d = mid;
      lo = mid + 1;
    } else {
      hi = mid - 1;
    }
  }
  const TrsvDom &D = st.d[d];
  if (D.active && !*D.active) return;   // (fused batch) a cell whose Arnoldi steps are paused
  const int blk = vb - (kind == 0 ? D.first_block : kind == 1 ? D.first_z : D.first_bulk);
  const int64_t ld = D.ld;
  const C *__restrict__ F = (const C *)D.F;
  if (kind == 0) {
    // (1) row r of block j, one per wave: every load is issued before the
    // barrier (the row's rhs, its entries in block j-2, row r of G_j, its
    // chunk sums, z_{j-2} and r_{j-1} for shared memory)
    const int cb0 = D.cb0, cm = D.cm, pm = D.pm, nb0 = D.nb0, nm = D.nm;
    const int r = 16 * blk + wave;
    const int ic = nb0 + clampi(r, nm - 1);
    dz *zo = sm, *zn = sm + NV * kTrsvNB;
    TrsvVec<NV> po, pn;
    po.fetch([&](int q) { return D.sol[q] + cb0; }, cm);
    pn.fetch([&](int q) { return D.rin + q * kTrsvNB; }, pm);
    dz rv[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) rv[q] = D.rhs[q][ic];
    // (kept in the factor type until used: registers bound the occupancy)
    const int gld = D.gld;
    const C *__restrict__ G = (const C *)D.G + (int64_t)clampi(r, kTrsvNB - 1) * gld;
    C fo[kTrsvCol], fg[kTrsvCol];
#pragma unroll
    for (int c = 0; c < kTrsvCol; ++c) {
      fo[c] = F[(int64_t)ic * ld + cb0 + clampi(lane + 64 * c, cm - 1)];
      fg[c] = G[gld > 0 ? lane + 64 * c : 0];
    }
#pragma unroll
    for (int c = 0; c < kTrsvCol; ++c) {
      if (!(lane + 64 * c < cm)) fo[c] = cx<C>::make(0, 0);
      if (!(lane + 64 * c < pm)) fg[c] = cx<C>::make(0, 0);
    }
    // chunk sums of row r: lane l takes chunks l and l + 64 (bst <= 128; the
    // second only for domains of more than 64 chunks, under a uniform branch)
    dz bs[NV];
    const int bst = D.bst, nci = D.nci;
    const dz *bp = D.bsum_in + (int64_t)clampi(r, kTrsvNB - 1) * bst;
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      const dz b0 = bp[(int64_t)q * kTrsvNB * bst + clampi(lane, bst - 1)];
      bs[q] = lane < nci ? b0 : mk(0, 0);
    }
    if (nci > 64) {
#pragma unroll
      for (int q = 0; q < NV; ++q) {
        const dz b1 = bp[(int64_t)q * kTrsvNB * bst + clampi(lane + 64, bst - 1)];
        bs[q] = bs[q] + (lane + 64 < nci ? b1 : mk(0, 0));
      }
    }
    po.store(zo, cm);
    pn.store(zn, pm);
    __syncthreads();
    // the chunk sums, then the updates of blocks j-2 and j-1, in that order
    dz rg[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      dz so = mk(0, 0), sn = mk(0, 0);
#pragma unroll
      for (int c = 0; c < kTrsvCol; ++c) cmac(so, to_dz(fo[c]), zo[q * kTrsvNB + lane + 64 * c]);
#pragma unroll
      for (int c = 0; c < kTrsvCol; ++c) cmac(sn, to_dz(fg[c]), zn[q * kTrsvNB + lane + 64 * c]);
      const dz sb = wave_sum_dpp(bs[q]);
      so = wave_sum_dpp(so);
      sn = wave_sum_dpp(sn);
      rg[q] = ((rv[q] - sb) - so) - sn;
    }
    if (lane == 0 && r < nm) {
#pragma unroll
      for (int q = 0; q < NV; ++q) D.rout[q * kTrsvNB + r] = rg[q];
    }
    return;
  }
  if (kind == 1) {
    // (2) row o of inv(T_{j-1,j-1}), one per wave, against r_{j-1}
    const int pb0 = D.pb0, pm = D.pm;
    const int o = 16 * blk + wave;
    dz *zn = sm;
    TrsvVec<NV> pn;
    pn.fetch([&](int q) { return D.rin + q * kTrsvNB; }, pm);
    const C *__restrict__ IV = (const C *)D.INV + (int64_t)clampi(o, pm - 1) * pm;
    C fi[kTrsvCol];
#pragma unroll
    for (int c = 0; c < kTrsvCol; ++c) fi[c] = IV[clampi(lane + 64 * c, pm - 1)];
#pragma unroll
    for (int c = 0; c < kTrsvCol; ++c)
      if (!(lane + 64 * c < pm)) fi[c] = cx<C>::make(0, 0);
    pn.store(zn, pm);
    __syncthreads();
    dz zq[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      dz a = mk(0, 0);
#pragma unroll
      for (int c = 0; c < kTrsvCol; ++c) cmac(a, to_dz(fi[c]), zn[q * kTrsvNB + lane + 64 * c]);
      zq[q] = wave_sum_dpp(a);
    }
    if (lane == 0 && o < pm) {
#pragma unroll
      for (int q = 0; q < NV; ++q) D.sol[q][pb0 + o] = zq[q];
    }
    return;
  }
  // (a) work item ch of the next block's row group rgp: one row per wave,
  // lane l holding columns l + 64 t of the item's KC columns; the item's
  // solutions are staged in shared memory (zero past the item's end, so
  // clamped factor reads add 0).  Each kTrsvSumCols columns give one chunk
  // sum: lane sums in column order, then the wave sum.
  static_assert(KC % kTrsvSumCols == 0 && kTrsvSumCols == 1024, "chunks of one pass of 1024 threads");
  const int b = blk;
  const int ch = b / D.nrg, rgp = b - ch * D.nrg;
  const int cs = D.bc0 + ch * KC;
  const int cn = min(KC, D.bc0 + D.bk - cs);
  const int sc0 = ch * (KC / kTrsvSumCols);   // the item's first chunk
  const int r = 16 * rgp + wave;
  const int i = D.br0 + clampi(r, D.brm - 1);
  constexpr int kPer = KC / 1024;
  dz zv[NV][kPer];
#pragma unroll
  for (int q = 0; q < NV; ++q)
#pragma unroll
    for (int u = 0; u < kPer; ++u) zv[q][u] = D.sol[q][cs + clampi(tid + 1024 * u, cn - 1)];
  constexpr int T = KC / 64;                                 // factor entries per lane
  constexpr int LB = sizeof(C) == 8 && NV == 1 ? 16 : 8;     // entries per batch of loads
  constexpr int NB = T / LB;
  constexpr int kBatchesPerSum = kTrsvSumCols / 64 / LB;
  static_assert(T % LB == 0 && (kTrsvSumCols / 64) % LB == 0, "whole batches per chunk");
  const C *__restrict__ row = F + (int64_t)i * ld + cs;
  C fa[LB];
#pragma unroll
  for (int u = 0; u < LB; ++u) fa[u] = row[clampi(lane + 64 * u, cn - 1)];
#pragma unroll
  for (int q = 0; q < NV; ++q)
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int t = tid + 1024 * u;
      sm[q * KC + t] = t < cn ? zv[q][u] : mk(0, 0);
    }
  __syncthreads();
  dz s[NV];
#pragma unroll
  for (int q = 0; q < NV; ++q) s[q] = mk(0, 0);
  const auto use = [&](const C(&f)[LB], int bt) {
#pragma unroll
    for (int u = 0; u < LB; ++u) {
      const int t = lane + 64 * (bt * LB + u);
      const dz fu = to_dz(f[u]);
#pragma unroll
      for (int q = 0; q < NV; ++q) cmac(s[q], fu, sm[q * KC + t]);
    }
    __builtin_amdgcn_sched_barrier(0);   // no hoisting of one batch's work into another's
  };
  // chunk h of the item done: every vector's wave sum, then lane 0's stores
  // (no vector's arithmetic moves past another's store branch)
  const auto flush = [&](int h) {
#pragma unroll
    for (int q = 0; q < NV; ++q) s[q] = wave_sum_dpp(s[q]);
    if (lane == 0 && r < D.brm && h * kTrsvSumCols < cn) {
#pragma unroll
      for (int q = 0; q < NV; ++q)
        D.bsum_out[(int64_t)q * kTrsvNB * D.bst + (int64_t)r * D.bst + sc0 + h] = s[q];
    }
#pragma unroll
    for (int q = 0; q < NV; ++q) s[q] = mk(0, 0);
  };
  // batch bt + 1 loads while batch bt is used (a rolled loop, so that the
  // compiler keeps two batches in registers rather than hoisting them all);
  // the last batch is used after the loop
#pragma unroll 1
  for (int bt = 0; bt < NB - 1; ++bt) {
    C fb[LB];
#pragma unroll
    for (int u = 0; u < LB; ++u) fb[u] = row[clampi(lane + 64 * ((bt + 1) * LB + u), cn - 1)];
    use(fa, bt);
    if ((bt + 1) % kBatchesPerSum == 0) flush(bt / kBatchesPerSum);
#pragma unroll
    for (int u = 0; u < LB; ++u) fa[u] = fb[u];
  }
  use(fa, NB - 1);
  flush(KC / kTrsvSumCols - 1);
}

#define VIE_TRSV_STEP(T, C, K)                                                                  \
  __global__ __launch_bounds__(1024) void k_trsv_step_##T##_k##K(TrsvStep st) {                \
    trsv_step_body<C, K, 1>(st, blockIdx.x);                                                  \
  }                                                                                           \
  __global__ __launch_bounds__(1024) void k_trsv_step2_##T##_k##K(TrsvStep st) {               \
    trsv_step_body<C, K, 2>(st, blockIdx.x);                                                  \
  }
VIE_TRSV_STEP(z, dz, 1024)
VIE_TRSV_STEP(z, dz, 2048)
VIE_TRSV_STEP(c, fz, 1024)
VIE_TRSV_STEP(c, fz, 2048)

// Every step of the triangular solves in one cooperative launch: the thread
// blocks share each step's work items (the same items the per-step launches
// give to their thread blocks) and meet at a grid barrier between steps,
// which orders one step's partial products before the next step's sums.
// All blocks run the same loops and reach every barrier.
template <typename C, int KC>
__device__ __forceinline__ void trsv_coop_body(const TrsvStep *__restrict__ plan, int nsteps) {
  cooperative_groups::grid_group grid = cooperative_groups::this_grid();
  for (int s = 0; s < nsteps; ++s) {
    const TrsvStep &st = plan[s];
    const int total = st.total_blocks;
    for (int vb = blockIdx.x; vb < total; vb += gridDim.x) {
      __syncthreads();   // the previous item's shared memory is free
      trsv_step_body<C, KC, 1>(st, vb);
    }
    grid.sync();
  }
}

// One step of a batch's fused triangular solves (one vector per cell): the
// step's domains of every cell, read from device memory.
struct TrsvStepDev {
  const TrsvDom *d;
  int ndom, lower, chain_blocks, z_end;
};
#define VIE_TRSV_STEPD(T, C)                                                                      \
  __global__ __launch_bounds__(1024) void k_trsv_stepd_##T(const TrsvDom *doms, int ndom, int lower,   \
                                                            int chain_blocks, int z_end) {             \
    const TrsvStepDev st{doms, ndom, lower, chain_blocks, z_end};                                     \
    trsv_step_body<C, kTrsvSumCols, 1, TrsvStepDev>(st, blockIdx.x);                             \
  }
VIE_TRSV_STEPD(z, dz)
VIE_TRSV_STEPD(c, fz)

#define VIE_TRSV_COOP(T, C, K)                                                                  \
  __global__ __launch_bounds__(1024) void k_trsv_coop_##T##_k##K(const TrsvStep *plan, int nsteps) { \
    trsv_coop_body<C, K>(plan, nsteps);                                                       \
  }
VIE_TRSV_COOP(z, dz, 1024)
VIE_TRSV_COOP(z, dz, 2048)
VIE_TRSV_COOP(c, fz, 1024)
VIE_TRSV_COOP(c, fz, 2048)

}  // namespace vie
