// Gradient contraction.  For one block, with e, g and Q = L^{-T} [0; I_b] from the
// adjoint solves (e, g, then the columns of Q, column stride nA):
//   dl_i/dtheta_k = 1/2 sum_ab M_ab dSigma_ab/dtheta_k,
//   M = e g^T + g e^T + g g^T - Q Q^T,
// with dSigma recomputed from the scaled coordinates:
//   d/dlog beta_k: sigma^2 (-rho'(r)/r) s_k^2,  d/dlog sigma^2: sigma^2 rho(r),
//   d/dlog tau^2: tau^2 on the diagonal.
//
// The tiles of the lower triangle are taken one at a time: Q Q^T of a tile on MFMA
// (five at b = 20 points), then its four entries per lane on the vector ALU, about
// 75 FP64 instructions each at d = 10, which is what bounds the kernel (FP64 MFMA
// and vector instructions share the SIMD's pipe).  Nothing but the d + 2 sums
// lives across tiles, so three blocks share a compute unit.  A wave owns tile rows
// i, dealt so that every wave has the same number of tiles: its lanes keep the
// coordinates of point 16 i + c, the other four points of an entry are read from
// LDS by all 16 lanes of a group at once, and the squared differences of an entry
// stay in registers between the distance and the derivatives.  The first columns
// of Q are staged in LDS, as many as leave the occupancy; the rest is read from the
// adjoint buffer.  n = 2e5, m = 200, d = 10: 4.7 -> 1.4 ms FP64 and
// 3.9 -> 0.95 ms FP32 (all tiles of a block in registers, one block a unit, before);
// 2,400 blocks of m = 400: 3.3 -> 1.6 ms.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "block_device.h"
#include "sbv_internal.h"

namespace sbv {

constexpr int kCW = 4;  // waves per workgroup

// The first lane's value, known to be uniform (scalar registers).
__device__ __forceinline__ double uniform(double v) {
  return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                          __builtin_amdgcn_readfirstlane(__double2loint(v)));
}
__device__ __forceinline__ float uniform(float v) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// Derivative factors of the covariance: rho sigma^2 = (p0 + r (p1 + r (p2 + r p3))) e^{-r}
// and sigma^2 (-rho'(r)/r) = (h0 + r (h1 + r h2)) e^{-r}, the latter over r for nu = 1/2.
template <typename T>
struct CovGrad {
  T p0, p1, p2, p3, h0, h1, h2;
  __device__ CovGrad(T s2v, int two_nu) {
    const T s2 = uniform(s2v);
    p0 = s2;
    p1 = two_nu >= 3 ? s2 : T(0);
    p2 = two_nu == 5 ? s2 * T(1.0 / 3.0) : (two_nu == 7 ? s2 * T(0.4) : T(0));
    p3 = two_nu == 7 ? s2 * T(1.0 / 15.0) : T(0);
    // (nu = 1/2: over r, by the caller)
    h0 = two_nu == 5 ? s2 * T(1.0 / 3.0) : (two_nu == 7 ? s2 * T(0.2) : s2);
    h1 = two_nu >= 5 ? h0 : T(0);
    h2 = p3;
  }
};

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 8; o >= 1; o >>= 1) v += __shfl_xor(v, o, 16);
  return rows_sum(v);
}

// The rows of tiles dealt to one wave.  NU1: nu = 1/2, whose -rho'(r)/r is
// e^{-r} / r (0 at r = 0, where it meets a zero difference).
template <typename T, int D, bool NU1>
__device__ __forceinline__ void contract_rows(const typename ZV<T>::v* zs, const T* ev, const T* gv, const T* qs,
                                              const __attribute__((address_space(1))) T* src, const T* tab,
                                              const CovGrad<T>& cov, T tau2, int wave, int lane, int nt, int nA,
                                              int bi, int ps, int nql, int nq,
                                              double (&gacc)[(D + kOV<T> - 1) / kOV<T> * kOV<T>], double& gs,
                                              double& gt) {
  typedef typename MF<T>::acc acc_t;
  typedef typename ZV<T>::v zv;
  constexpr int NV = (D + kOV<T> - 1) / kOV<T>, DP = NV * kOV<T>;
  constexpr int kAtOnce = 2;  // entries of a lane in flight (registers)
  const int g = lane >> 4, c = lane & 15, np = kTile * nt;
      for (int s = 0; s * kCW < nt; ++s) {
        const int i = nt - 1 - kCW * s - ((s & 1) ? kCW - 1 - wave : wave);
        if (i < 0) continue;
        const int pb = kTile * i + c;
        T zb[DP];
#pragma unroll
        for (int e = 0; e < NV; ++e) {
          const zv v = zs[np * e + pb];
#pragma unroll
          for (int u = 0; u < kOV<T>; ++u) zb[kOV<T> * e + u] = v[u];
        }
        const T eb = ev[pb], gb = gv[pb], sb = eb + gb;
        for (int j = 0; j <= i; ++j) {
          acc_t P = {T(0), T(0), T(0), T(0)};
          const T* qa = qs + ps * g + kTile * j + c;
          const T* qb = qs + ps * g + pb;
          for (int q = 0; q < nql; ++q) P = MF<T>::mma(qa[4 * ps * q], qb[4 * ps * q], P);
          for (int q = nql; q < nq; ++q) {
            const int col = 4 * q + g, ra = kTile * j + c;
            const bool in = col < bi;
            const int64_t at = (int64_t)(2 + min(col, bi - 1)) * nA;
            const T va = src[at + min(ra, nA - 1)], vb = src[at + min(pb, nA - 1)];
            P = MF<T>::mma(in && ra < nA ? va : T(0), in && pb < nA ? vb : T(0), P);
          }
          const double half = i == j ? 0.5 : 1.0;  // 1/2 of every entry; off the diagonal it counts twice
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const int pa = kTile * j + MF<T>::row(g, t);
            const T ea = ev[pa], ga = gv[pa];
            T ds[DP], r2 = kTinyR2<T>;
#pragma unroll
            for (int e = 0; e < NV; ++e) {
              const zv df = zs[np * e + pa] - *reinterpret_cast<const zv*>(&zb[kOV<T> * e]);
#pragma unroll
              for (int u = 0; u < kOV<T>; ++u) {
                ds[kOV<T> * e + u] = df[u] * df[u];
                r2 += ds[kOV<T> * e + u];
              }
            }
            const T r = fmin(c_sqrt(r2), ExpTable<T>::end), ex = ExpTable<T>::exp_neg(r, tab);
            const T M = fma(ea, gb, fma(ga, sb, -P[t]));
            const T rho = fma(r, fma(r, fma(r, cov.p3, cov.p2), cov.p1), cov.p0) * ex;
            T h = fma(r, fma(r, cov.h2, cov.h1), cov.h0) * ex;
            if constexpr (NU1) h = r > T(1e-30) ? h / r : T(0);
            const double wm = half * (double)M, f = wm * (double)h;
#pragma unroll
            for (int k = 0; k < DP; ++k) gacc[k] += f * (double)ds[k];
            gs += wm * (double)rho;
            if (i == j && pa == pb) gt += wm * (double)tau2;
            if (t % kAtOnce == kAtOnce - 1) __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
}

// D: dimensions held (d <= D, the rest zero).  Dynamic LDS: coordinates (vectors of
// kOV dimensions, 16 nt points per vector row), e, g, then qcols columns of Q.
template <typename T, int D, int OCC>
__global__ __launch_bounds__(kCW * 64, OCC) void k_block_contract(const SetDesc* __restrict__ sets,
                                                                  const double* __restrict__ theta,
                                                                  const WorkItem* __restrict__ items,
                                                                  const int* __restrict__ count, int qcols) {
  typedef typename ZV<T>::v zv;
  constexpr int NV = (D + kOV<T> - 1) / kOV<T>, DP = NV * kOV<T>, NTHR = kCW * 64;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ double red[kCW][kMaxDim + 2];
  __shared__ double isc[kMaxDim];
  __shared__ T tab[ExpTable<T>::n];
  zv* const zs = reinterpret_cast<zv*>(smem_raw);
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  if (tid < ExpTable<T>::n) tab[tid] = ExpTable<T>::entry(tid);
  const int total = *count;
  for (int it = blockIdx.x; it < total; it += gridDim.x) {
    const WorkItem w = items[it];
    const SetDesc S = sets[w.set];
    const int d = __builtin_amdgcn_readfirstlane(S.d), two_nu = __builtin_amdgcn_readfirstlane(S.two_nu);
    const double* th = theta + S.theta_off;
    const int b0 = S.bptr[w.block], b1 = S.bptr[w.block + 1];
    const int64_t n0 = S.nptr[w.block], n1 = S.nptr[w.block + 1];
    const int mi = __builtin_amdgcn_readfirstlane((int)(n1 - n0)), bi = __builtin_amdgcn_readfirstlane(b1 - b0);
    const int nA = mi + bi, nt = (nA + kTile - 1) / kTile, np = nt * kTile;
    // column stride of Q in LDS: the four column groups of an operand read fall on
    // different banks
    constexpr int kS = 32 * 8 / (int)sizeof(T);
    const int ps = np + (kTile - np % kS + kS) % kS;
    T* const ev = reinterpret_cast<T*>(zs + NV * np);
    T* const gv = ev + np;
    T* const qs = gv + np;
    const auto src = as_global(reinterpret_cast<const T*>(S.qbuf)) + S.qoff[w.block];
    if (tid < d) isc[tid] = exp(-th[tid]);
    const CovGrad<T> cov(T(exp(th[d])), two_nu);
    const T tau2 = T(exp(th[d + 1]));
    __syncthreads();
    for (int p = tid; p < np; p += NTHR) {
      const bool real = p < nA;
      const int pos = !real ? b0 : p < mi ? as_global(S.nidx)[n0 + p] : b0 + (p - mi);
      const auto xr = as_global(S.X) + (int64_t)pos * d;
      double x[DP];
#pragma unroll
      for (int e = 0; e < DP; ++e) x[e] = xr[min(e, d - 1)];
#pragma unroll
      for (int e = 0; e < DP; e += kOV<T>) {
        zv v;
#pragma unroll
        for (int u = 0; u < kOV<T>; ++u) v[u] = (real && e + u < d) ? T(x[e + u] * isc[min(e + u, d - 1)]) : T(0);
        zs[np * (e / kOV<T>) + p] = v;
      }
      ev[p] = real ? src[p] : T(0);
      gv[p] = real ? src[nA + p] : T(0);
    }
    const int nq = (bi + 3) / 4;                  // groups of four columns (the last one zero padded)
    const int nql = min(nq, qcols / 4);           // those in LDS
    for (int e = tid; e < 4 * nql * np; e += NTHR) {
      const int col = e / np, r = e - col * np;
      qs[ps * col + r] = (r < nA && col < bi) ? src[(int64_t)(2 + col) * nA + r] : T(0);
    }
    __syncthreads();
    double gacc[DP], gs = 0.0, gt = 0.0;
#pragma unroll
    for (int k = 0; k < DP; ++k) gacc[k] = 0.0;
    if (two_nu == 1)
      contract_rows<T, D, true>(zs, ev, gv, qs, src, tab, cov, tau2, wave, lane, nt, nA, bi, ps, nql, nq, gacc, gs, gt);
    else
      contract_rows<T, D, false>(zs, ev, gv, qs, src, tab, cov, tau2, wave, lane, nt, nA, bi, ps, nql, nq, gacc, gs, gt);
    // fixed-order sums: lanes, then waves
#pragma unroll
    for (int k = 0; k < DP; ++k) {
      const double v = wave_sum(gacc[k]);
      if (k < kMaxDim && lane == 0) red[wave][k] = v;
    }
    gs = wave_sum(gs);
    gt = wave_sum(gt);
    __syncthreads();
    if (lane == 0) {
      red[wave][d] = gs;
      red[wave][d + 1] = gt;
    }
    __syncthreads();
    if (tid < d + 2) {
      double v = 0.0;
#pragma unroll
      for (int wv = 0; wv < kCW; ++wv) v += red[wv][tid];
      S.gradb[(int64_t)w.block * (d + 2) + tid] = v;
    }
    __syncthreads();
  }
}

// Columns of Q in LDS: as many as let `occ` workgroups share a compute unit's 160
// KB (static arrays aside), at most 32.
template <typename T, int D, int OCC>
static hipError_t launch_c(int grid, int max_joint, const SetDesc* sets, const double* theta, const WorkItem* items,
                           const int* count, hipStream_t s) {
  constexpr int NV = (D + kOV<T> - 1) / kOV<T>;
  constexpr int kS = 32 * 8 / (int)sizeof(T);
  const int nt = (max_joint + kTile - 1) / kTile, np = nt * kTile;
  const size_t base = (size_t)np * (16 * NV + 2 * sizeof(T));
  const size_t col = sizeof(T) * (np + kS);
  int q = 0;
  for (int occ = OCC; occ >= 1; --occ) {
    const size_t cap = 160 * 1024 / occ - 2048;
    if (base + 8 * col > cap && occ > 1) continue;
    q = base < cap ? (int)std::min<size_t>(32, (cap - base) / col / 4 * 4) : 0;
    break;
  }
  hipLaunchKernelGGL((k_block_contract<T, D, OCC>), dim3(grid), dim3(kCW * 64), base + q * col, s, sets, theta, items,
                     count, q);
  return hipGetLastError();
}

hipError_t launch_contract(int prec, int max_joint, int grid, int dmax, const SetDesc* sets, const double* theta,
                           const WorkItem* items, const int* count, hipStream_t s) {
  if (grid <= 0) return hipSuccess;
  if (dmax < 1 || dmax > kMaxDim || max_joint < 1 || max_joint > kTile * (kLargeNTM + kMaxPrefix))
    return hipErrorInvalidValue;
#define SBV_CALL(T, D, O) launch_c<T, D, O>(grid, max_joint, sets, theta, items, count, s)
  if (prec == 0) return dmax <= 4 ? SBV_CALL(double, 4, 3) : dmax <= 10 ? SBV_CALL(double, 10, 3) : SBV_CALL(double, 20, 2);
  return dmax <= 4 ? SBV_CALL(float, 4, 4) : dmax <= 12 ? SBV_CALL(float, 12, 4) : SBV_CALL(float, 20, 3);
#undef SBV_CALL
}

}  // namespace sbv
