// Left-looking block kernel: the joint Cholesky factorisation of one block's
// covariance with the rows of 16x16 tiles owned by waves.
//
// A workgroup computes the block term of Alg. 5 in one pass over the joint set A =
// J_i u B_i (conditioning points first): it gathers the scaled coordinates (Sec. 4.4
// Eq. (scale)) and the observations, builds Sigma_A = sigma^2 rho(r) + tau^2 I (Eq.
// (maternkernel)) and factors Sigma_A = L L^T.  The leading m_i x m_i part of L is
// Alg. 5's POTRF(Sigma_con), the off-diagonal part its TRSM(Sigma_cross) transposed
// and the trailing part POTRF(Sigma_con - Sigma_cor); z = L^{-1} [y_J; y_B] is its
// TRSVs and GEMV, and the block's own pivots and z_k give
//   l_i = -1/2 (sum z_k^2 + 2 sum log L_kk + b_i log 2 pi),
// accumulated in FP64.
//
// The joint set A = J u B of a block (conditioning points first) is cut into
// nt = ceil(nA / 16) tile rows.  Column k of the factor is built from
//   A_ik = Sigma_ik - sum_{j<k} L_ij L_kj^T      (rows i >= k),
//   L_kk = chol(A_kk),  L_ik = A_ik L_kk^{-T},
// so a covariance tile is generated when its column is reached, straight into
// the accumulator of its update, and a finished tile of L is only read until
// its row is eliminated.  At step k (nt - k) k tiles are alive, at most a
// quarter of nt^2 (49 of 105 tiles at nt = 14, where a right-looking
// factorisation keeps all 105): two blocks share a compute unit and one
// block's serial diagonal factorisations run beside the other's updates.
//
// Wave w owns the tile rows nt-1-w, nt-1-w-NW, .. (slots 0, 1, ..: the long late
// rows are dealt first).  A tile of L is kept as G = L^T in the accumulator
// layout, where register q of lane (g, c) = (l / 16, l % 16) holds L[c][g + 4q].
// That is the B operand of every product the tile's own row takes part in, so an
// update reads only row k's tiles from LDS (the A operand, published by row k's
// owner), one read per tile for all rows of the wave.  Accumulators hold -A_ik^T,
// so that an update is a plain MFMA accumulation; the column solve G_ik =
// L_kk^{-1} A_ik^T takes its B operand from the accumulator itself.  A diagonal
// tile A_kk needs only its own row, whose owner keeps both operands in registers:
// it is generated and updated with the columns before k - 1 one step ahead, while
// the owner of row k - 1 factors, and takes one product more before its own
// factorisation.  The forward solve z = L^{-1} y rides along: every owner adds
// L_ik z_k to its rows' running sums.
//
// Two barriers per step: row k published | factorisation of tile (k, k) by its
// owner, column k generated and updated, tile (k+1, k+1) prepared | column solve.
// With a part of the factor in memory (tile_map) every diagonal tile is generated at
// the start and updated by each column solve of its row instead, in the same order.
//
// What bounds it (FP64, 14 tiles, two blocks per unit): of 250,000 cycles a SIMD's
// two waves issue matrix instructions in 29 % and vector instructions in 28 %, which
// do not overlap (an FP64 MFMA holds the vector pipe for its 64 cycles); half of a
// wave's time is spent at the two barriers and behind LDS reads.  Measured per
// evaluation, against the right-looking kernel with all tiles in registers and one
// block per unit: n = 1e6, m = 200 17.3 -> 10.1 ms; n = 2e4, m = 60 153 -> 52 us; n =
// 2e5, m = 200 in FP32 3.26 -> 1.45 ms; n = 1e5, m = 400 (a two-kernel path then) 12.7 ->
// 5.45 ms; value and gradient n = 2e5, m = 200 10.6 -> 4.13 ms.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>
#include <type_traits>

#include "block_device.h"
#include "sbv_internal.h"

namespace sbv {

// Register file of one wave's tiles, in tiles.  Tile (slot s, column j) is
// written at the end of step j and dead after step maxrow(s) = NTM - 1 - s NW
// (the wave's row of that slot is eliminated by then); the accumulator of slot s
// is used up to that step too.  Later columns of the long rows take over the
// registers of the short ones.
//
// CAP > 0 (large blocks): CAP tiles in all, and every slot keeps its diagonal tile
// from the first step on.  Slot s holds its columns j < res[s], which are read the
// most often, in registers; the later ones go to memory.  res is chosen greedily by
// the number of reads a register saves.
template <int NTM, int NW>
struct TileMap {
  static constexpr int NS = (NTM + NW - 1) / NW;
  int at[NS][NTM];
  int acc[NS];
  int dg[NS];
  int res[NS];
  int n;
  int ord[NS];   // slots by res, ascending
  int rank[NS];  // a slot's place in ord
  int fetch;     // tiles of one row in memory, per wave
};
template <int NTM, int NW, int CAP = 0>
constexpr TileMap<NTM, NW> tile_map() {
  TileMap<NTM, NW> m{};
  constexpr int NS = TileMap<NTM, NW>::NS;
  int dead[(NTM + 2) * NS] = {};  // step after which a register is free again
  for (int s = 0; s < NS; ++s) {
    m.acc[s] = m.n;
    dead[m.n++] = NTM - 1 - s * NW;
  }
  for (int s = 0; s < NS && CAP; ++s) {
    m.dg[s] = m.n;
    dead[m.n++] = NTM - 1 - s * NW;
  }
  for (int s = 0; s < NS; ++s) m.res[s] = CAP ? 0 : NTM;
  while (CAP) {
    int best = -1;
    for (int s = 0; s < NS; ++s) {
      const int last = NTM - 1 - s * NW;
      if (m.res[s] >= last || (best >= 0 && last - m.res[s] <= NTM - 1 - best * NW - m.res[best])) continue;
      bool fits = true;
      for (int t = 0; t < NTM; ++t) {
        int live = 0;
        for (int u = 0; u < NS; ++u) {
          const int r = m.res[u] + (u == s ? 1 : 0);
          if (NTM - 1 - u * NW >= t) live += 2 + (t + 1 < r ? t + 1 : r);
        }
        fits = fits && live <= CAP;
      }
      if (fits) best = s;
    }
    if (best < 0) break;
    ++m.res[best];
  }
  for (int s = 0; s < NS; ++s) {
    const int out = NTM - 1 - s * NW - m.res[s];
    for (int u = 0; u < NS; ++u) m.rank[s] += m.res[u] < m.res[s] || (m.res[u] == m.res[s] && u < s) ? 1 : 0;
    m.ord[m.rank[s]] = s;
    if ((out + NW - 1) / NW > m.fetch) m.fetch = (out + NW - 1) / NW;
  }
  for (int j = 0; j < NTM; ++j)
    for (int s = 0; s < NS; ++s) {
      m.at[s][j] = -1;
      const int last = NTM - 1 - s * NW;  // largest row of the slot: tiles j < last
      if (j >= last || j >= m.res[s]) continue;
      int r = 0;
      while (r < m.n && dead[r] > j) ++r;
      if (r == m.n) ++m.n;
      m.at[s][j] = r;
      dead[r] = last;
    }
  return m;
}

// Place of wave w among the NW rows of slot s (0: the largest).  With four waves
// the long and the short rows are paired so that every wave has about the same
// number of tiles and products (rows 13, 6, 4 / 12, 7, 5 / 11, 9, 3, 1 / 10, 8, 2, 0
// at nt = 14), and no wave owns two consecutive rows (the owner of row k + 1
// prepares its diagonal tile while the owner of row k factors).
template <int NW>
__device__ __forceinline__ int deal(int s, int w) {
  if (NW >= 8) return s == 1 || s == 2 ? NW - 1 - w : w;
  if (NW != 4 || s == 0) return w;
  return ((s & 1 ? 0x1023 : 0x3201) >> (4 * w)) & 3;
}

// Logical row of the MFMA output: register t of lane group g holds row g + 4t
// in both precisions.  FP64 does so by itself; FP32 outputs row 4g + t, so its A
// operands are read with the rows permuted (lane c takes row (c / 4) + 4 (c % 4)).
template <typename T>
__device__ __forceinline__ int a_lane(int lane) {
  return sizeof(T) == 8 ? lane : ((lane & 48) | ((lane >> 2) & 3) | ((lane & 3) << 2));
}

// Operand tiles in LDS: 16-byte vectors of kOV registers per lane, lane after lane.
template <typename T>
__device__ __forceinline__ void put_operand(T* tile, int lane, const T (&v)[4]) {
  typedef typename ZV<T>::v zv;
#pragma unroll
  for (int p = 0; p < 4 / kOV<T>; ++p) {
    zv x;
#pragma unroll
    for (int e = 0; e < kOV<T>; ++e) x[e] = v[kOV<T> * p + e];
    *reinterpret_cast<zv*>(tile + 64 * kOV<T> * p + kOV<T> * lane) = x;
  }
}
template <typename T>
__device__ __forceinline__ void get_operand(const T* tile, int lane, T (&v)[4]) {
  typedef typename ZV<T>::v zv;
#pragma unroll
  for (int p = 0; p < 4 / kOV<T>; ++p) {
    const zv x = *reinterpret_cast<const zv*>(tile + 64 * kOV<T> * p + kOV<T> * lane);
#pragma unroll
    for (int e = 0; e < kOV<T>; ++e) v[kOV<T> * p + e] = x[e];
  }
}
// A 16-vector stored so that lane group g reads its entries g + 4q as vectors.
__device__ __forceinline__ int vec_at(int r) { return 4 * (r & 3) + (r >> 2); }
template <typename T>
__device__ __forceinline__ void get_vec(const T* vec, int g, T (&v)[4]) {
  typedef typename ZV<T>::v zv;
#pragma unroll
  for (int p = 0; p < 4 / kOV<T>; ++p) {
    const zv x = *reinterpret_cast<const zv*>(vec + 4 * g + kOV<T> * p);
#pragma unroll
    for (int e = 0; e < kOV<T>; ++e) v[kOV<T> * p + e] = x[e];
  }
}

// Elimination of a 16x16 tile as L D L^T, held row by row: lane (r, .) has row r
// of A in a[] and W[r][g + 4q], W = I at first, in w[q].  On return a[c], c <= r,
// of lane r holds L[r][c] D_c (L unit lower) and w[q] the entries g + 4q of row r
// of L^{-1}.  Step J takes the multiple A[r][J] / D_J of row J from every row r > J of
// A and W: one reciprocal, one multiplier per row and one fused multiply-add per
// register, row J's value read from lane J of each 16-lane row by the DPP source
// of v_fmac.  Square roots are left to the caller (one per row, not per step).
//
// The order of a step is fixed because the factorisation is a serial chain beside
// another wave: an FP64 MFMA of the other block's wave on this SIMD holds the
// vector pipe for 64 cycles, and one slips in whenever this wave, though it has
// the higher priority, has no instruction ready.  In the compiler's order, with
// wait states around every DPP read, a tile took 3.0k cycles alone and 7.4k beside
// another block.  So the chain of step J + 1 (pivot column, pivot p, reciprocal r
// to 2^-24, e = 1 - p r, m0 = -A r, m = m0 (1 + e + e^2)) is interleaved with the
// updates of step J, which stand between a DPP read and the write of its register
// (two wait states) and between the reciprocal and its use.  Each statement opens
// with instructions that read no DPP source, for whatever the compiler puts
// before it.
#define SBV_DPP " row_newbcast:%c[j] row_mask:0xf bank_mask:0xf\n\t"
#define SBV_U(FM, x) FM " %[" x "], %[" x "], %[m]" SBV_DPP
#define SBV_IF(cond, text) ".if " cond "\n\t" text ".endif\n\t"
#define SBV_A(FM, c) SBV_IF(#c " > %c[j] + 1", SBV_U(FM, "a" #c))
// first half of step J: its multipliers, the next pivot's column, pivot and reciprocal
#define SBV_ELIM_HEAD(FM, MOV, RCP, FMA, ONE)                                                                       \
  asm(FMA " %[m], %[f], %[m0], %[m0]\n\ts_nop 0\n\t" SBV_U(FM, "n") SBV_U(FM, "w0") SBV_A(FM, 15)                    \
          SBV_IF("%c[j] > 13", SBV_U(FM, "w1")) MOV                                                                 \
      " %[p], %[n] row_newbcast:%c[j1] row_mask:0xf bank_mask:0xf\n\t"                                              \
      "s_lshl_b64 %[eq], %[eq], 1\n\t" RCP " %[r], %[p]\n\ts_andn2_b64 %[ab], %[ab], %[eq]\n\t"                       \
          SBV_IF("(%c[j] > 3) && (%c[j] < 14)", SBV_U(FM, "w1")) SBV_IF("%c[j] > 7", SBV_U(FM, "w2"))               \
              SBV_IF("%c[j] > 11", SBV_U(FM, "w3")) SBV_A(FM, 14) SBV_A(FM, 13) SBV_A(FM, 12) SBV_A(FM, 11) FMA     \
      " %[e], -%[p], %[r], " ONE "\n\t" SBV_A(FM, 10) SBV_A(FM, 9)                                                  \
      : [m] "=&v"(m), [n] "+v"(a[J + 1]), [w0] "+v"(w[0]), [w1] "+v"(w[1]), [w2] "+v"(w[2]), [w3] "+v"(w[3]),       \
        [a9] "+v"(a9), [a10] "+v"(a10), [a11] "+v"(a11), [a12] "+v"(a12), [a13] "+v"(a13), [a14] "+v"(a14),         \
        [a15] "+v"(a15), [p] "=&v"(p), [r] "=&v"(r), [e] "=&v"(e), [eq] "+s"(eq), [ab] "+s"(ab)                     \
      : [f] "v"(f), [m0] "v"(m0), [j] "i"(J), [j1] "i"(J + 1)                                                       \
      : "scc")
// second half: the next multipliers' first factor and correction, the other updates
#define SBV_ELIM_TAIL(FM, MUL, CORR)                                                                                \
  asm(MUL " %[m0], %[am], -%[r]\n\t" CORR SBV_A(FM, 8) SBV_A(FM, 7) SBV_A(FM, 6) SBV_A(FM, 5) SBV_A(FM, 4)           \
          SBV_A(FM, 3) SBV_A(FM, 2)                                                                                 \
      : [m0] "=&v"(m0), [f] "=&v"(f), [a2] "+v"(a[2]), [a3] "+v"(a[3]), [a4] "+v"(a[4]), [a5] "+v"(a[5]), [a6] "+v"(a[6]),    \
        [a7] "+v"(a[7]), [a8] "+v"(a[8])                                                                                \
      : [m] "v"(m), [am] "v"(am), [r] "v"(r), [e] "v"(e), [j] "i"(J))

__device__ __forceinline__ double rcp_hw(double p) { return __builtin_amdgcn_rcp(p); }
__device__ __forceinline__ float rcp_hw(float p) { return __builtin_amdgcn_rcpf(p); }
// v in the lanes of the mask, 0 elsewhere.
__device__ __forceinline__ unsigned sel_u(unsigned v, unsigned long long mask) {
  unsigned x;
  asm("v_cndmask_b32_e64 %0, 0, %1, %2" : "=v"(x) : "v"(v), "s"(mask));
  return x;
}
__device__ __forceinline__ double sel(double v, unsigned long long mask) {
  const unsigned lo = sel_u((unsigned)__double2loint(v), mask), hi = sel_u((unsigned)__double2hiint(v), mask);
  return __hiloint2double((int)hi, (int)lo);
}
__device__ __forceinline__ float sel(float v, unsigned long long mask) {
  return __uint_as_float(sel_u(__float_as_uint(v), mask));
}

template <int J, typename T>
__device__ __forceinline__ void ldl_step(T (&a)[16], T (&w)[4], T f, T m0, unsigned long long eq,
                                         unsigned long long ab) {
  // (the head's columns up to J are operands but not touched; J + 1 is named by
  // itself, so its number goes to a stand-in)
  T m, p, r, e, am, no;
  T &a9 = J == 8 ? no : a[9], &a10 = J == 9 ? no : a[10], &a11 = J == 10 ? no : a[11], &a12 = J == 11 ? no : a[12],
    &a13 = J == 12 ? no : a[13], &a14 = J == 13 ? no : a[14], &a15 = J == 14 ? no : a[15];
  if constexpr (sizeof(T) == 8) {
    SBV_ELIM_HEAD("v_fmac_f64_dpp", "v_mov_b64_dpp", "v_rcp_f64_e32", "v_fma_f64", "1.0");
  } else {
    SBV_ELIM_HEAD("v_fmac_f32_dpp", "v_mov_b32_dpp", "v_rcp_f32_e32", "v_fma_f32", "1.0");
  }
  if constexpr (J < 14) {
    am = sel(a[J + 1], ab);
    if constexpr (sizeof(T) == 8) {
      SBV_ELIM_TAIL("v_fmac_f64_dpp", "v_mul_f64", "v_fma_f64 %[f], %[e], %[e], %[e]\n\t");
    } else {
      SBV_ELIM_TAIL("v_fmac_f32_dpp", "v_mul_f32_e64", "v_mov_b32_e32 %[f], %[e]\n\t");
    }
    ldl_step<J + 1>(a, w, f, m0, eq, ab);
  }
}
template <typename T>
__device__ __forceinline__ void ldl(T (&a)[16], T (&w)[4]) {
  const T piv = row_first(a[0]), r = rcp_hw(piv), e = fma(-piv, r, T(1));
  unsigned long long eq = 0x0001000100010001ull, ab = ~eq;  // lanes r = J and r > J
  __asm__ volatile("" : "+s"(eq), "+s"(ab));
  ldl_step<0>(a, w, sizeof(T) == 8 ? fma(e, e, e) : e, sel(a[0], ab) * -r, eq, ab);
}

// Row stride of the diagonal tile in LDS (16-byte rows, two rows never on the
// same banks).
template <typename T>
constexpr int kDg = 16 + kOV<T>;

// Negated covariance function with its constants folded: -sigma^2 p(r) e^{-r}, in
// FP64 for both precisions.  EXACT: to the last digits of FP64; otherwise to 2^-38, far below FP32's.
struct Cov {
  double p0, p1, p2, p3;
  __device__ Cov(double sigma2, int two_nu) {
    p0 = -sigma2;
    p1 = two_nu >= 3 ? p0 : 0.0;
    p2 = two_nu == 5 ? p0 * (1.0 / 3.0) : (two_nu == 7 ? p0 * 0.4 : 0.0);
    p3 = two_nu == 7 ? p0 * (1.0 / 15.0) : 0.0;
  }
  template <bool EXACT>
  __device__ __forceinline__ double eval(double r2, const double* tab) const {
    const double r = c_sqrt<EXACT>(r2);  // (NaN where r2 overflows: it has to reach the pivots)
    return fma(r, fma(r, fma(r, p3, p2), p1), p0) *
           ExpTable<double>::exp_neg<EXACT>(fmin(r, ExpTable<double>::end), tab);
  }
};

// Negated covariance tiles (row[n], k), n < N, in the accumulator layout of the
// transposed tile: register t of lane (g, c) is the entry of points 16 k + g +
// 4t and 16 row[n] + c.  Coordinates (FP64) are stored as 16-byte vectors of two
// dimensions, P points per vector row, so that every read has a constant offset
// (reading the next vector while one is used spills: 8325 against 8060 us, 14 tiles).
// The four points of tile k are read once for all N rows.  Only the last tile row and
// column (padding: identity) and diagonal tiles (nugget) need their entries looked at.
// NAT: rows in the MFMA output's own order (diagonal tiles, whose A operand is
// the unpermuted register).
template <typename T, int N, int P, bool NAT = false>
__device__ __forceinline__ void gen_tiles(const double* z, const double* tab, int nv, int lane, int k, const int (&row)[N],
                                          int nt, int nA, const Cov& cov, double tau2, double (&v)[N][4]) {
  typedef typename ZV<double>::v zv;
  const int g = lane >> 4, c = lane & 15;
  auto prow = [](int g, int t) { return NAT ? MF<T>::row(g, t) : g + 4 * t; };
  const zv* za = reinterpret_cast<const zv*>(z) + kTile * k + prow(g, 0);
  const zv* zb[N];
  zv a[4], b[N];
  auto load = [&]() {
#pragma unroll
    for (int t = 0; t < 4; ++t) a[t] = za[prow(0, t)];
#pragma unroll
    for (int n = 0; n < N; ++n) b[n] = zb[n][0];
  };
#pragma unroll
  for (int n = 0; n < N; ++n) {
    zb[n] = reinterpret_cast<const zv*>(z) + kTile * row[n] + c;
#pragma unroll
    for (int t = 0; t < 4; ++t) v[n][t] = kTinyR2<double>;
  }
  auto add = [&]() {
#pragma unroll
    for (int n = 0; n < N; ++n)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const zv df = a[t] - b[n];
#pragma unroll
        for (int x = 0; x < kOV<double>; ++x) v[n][t] += df[x] * df[x];
      }
  };
#pragma unroll 1
  for (int e = 0; e < nv; ++e) {
    load();
    add();
    za += P;
#pragma unroll
    for (int n = 0; n < N; ++n) zb[n] += P;
  }
#pragma unroll
  for (int n = 0; n < N; ++n) {
#pragma unroll
    for (int t = 0; t < 4; ++t) v[n][t] = cov.eval<sizeof(T) == 8>(v[n][t], tab);
    if (N > 1) __builtin_amdgcn_sched_barrier(0);  // (four entries in flight: registers)
  }
#pragma unroll
  for (int n = 0; n < N; ++n) {
    if (NAT) {
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (prow(g, t) == c) v[n][t] -= tau2;
    }
    if (row[n] == nt - 1) {  // (tile k = nt - 1 only meets row nt - 1)
      const int pb = kTile * row[n] + c;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int pa = kTile * k + prow(g, t);
        if (pa >= nA || pb >= nA) v[n][t] = pa == pb ? -1.0 : 0.0;
      }
    }
  }
}

// FP32 keeps what its rounding takes off a covariance entry and adds it when the
// running difference has shrunk to the size of the Schur complement.  That rounding
// was most of the error of the FP32 terms: without it the errors of value and
// gradient against FP64 are 0.4 times those of covariances rounded to FP32 (n = 1e5, d =
// 10, m = 200, tau^2 = 1e-3, sixteen datasets; emulated, 220 points, d = 5: 1.14e-3 of a
// term's 1.22e-3).  The price, n = 2e5, m = 200: 1088 + 377 us instead of 873 + 285 us.
template <typename T>
__device__ __forceinline__ T low_part(double v) {
  return sizeof(T) == 8 ? T(0) : T(v - (double)T(v));
}

// What a launch does with the factor.
//   kValue    the block's log-likelihood term
//   kSample   conditional simulation (and prediction): rows of J are solved, rows of
//             B take their innovations and emit y_B = L_BJ z_J + L' xi_B, with the
//             conditional variances (row sums of squares of L') when asked for
//   kAdjoint  the term, then the adjoint solves (adjoint_solves)
enum RowMode { kValue, kSample, kAdjoint };

// Tiles of L in memory (64 q + lane: register q of a G tile), by row.
__device__ __forceinline__ int tile_at(int i, int j) { return 256 * (i * (i + 1) / 2 + j); }
template <typename T, typename V>
__device__ __forceinline__ void tile_store(T* tile, int lane, const V& v) {
  const auto p = (__attribute__((address_space(1))) T*)tile;
#pragma unroll
  for (int q = 0; q < 4; ++q) p[64 * q + lane] = v[q];
}
template <typename T>
__device__ __forceinline__ void tile_load(const T* tile, int lane, T (&v)[4]) {
  const auto p = as_global(tile);
#pragma unroll
  for (int q = 0; q < 4; ++q) v[q] = p[64 * q + lane];
}

// Adjoint solves L^T X = R of one block, right-hand sides in chunks of kCB tile
// columns: column 0 is [z_J; 0] (its solution is e = [Sigma_J^{-1} y_J; 0]), column
// 1 is [0; z_B] (g = Q z_B) and column 2 + c the unit vector of row mi + c (the
// columns of Q = L^{-T} [0; I_b]).  Wave w owns the tile rows w, w + NW, .. of R and
// keeps them in registers; L is read once per chunk from memory, where the
// factorisation has left its tiles and minus the inverses of the diagonal ones.
// Step k uses X_k from LDS in R_j -= L_kj^T X_k; the owner of row k - 1 updates
// that row first, solves it and publishes X_{k-1} while the others update theirs:
// one barrier per step.  Bound by the chain of steps (update, solve, publish: about
// 4000 cycles of two blocks' waves), not by the products: 57,000 of a block's 340,000
// cycles at 14 tiles (FP64, two blocks per unit), 75,000 when every tile was requested
// and waited for by itself.
constexpr int kCB = 2;
template <int N, typename F>
__device__ __forceinline__ void unrolled_down(F&& f) {  // f(N - 1), .., f(0), as constants
  if constexpr (N > 0) {
    f(std::integral_constant<int, N - 1>{});
    unrolled_down<N - 1>(f);
  }
}
template <typename T>
constexpr int kXT = kTile * (kTile + kOV<T>);  // solution tile: columns of 16 rows, padded
template <typename T, int NTM, int NW>
__device__ __forceinline__ void adjoint_solves(T* xs, const T* yv, const T* lt, int lane, int wave, int nt, int mi,
                                               int nA, int bi, T* out) {
  typedef typename MF<T>::acc acc_t;
  typedef typename ZV<T>::v zv;
  constexpr int NS = (NTM + NW - 1) / NW, LD = kTile + kOV<T>;
  const int g = lane >> 4, c = lane & 15, ncol = bi + 2;
  // A operand of L_kj^T: rows 4g + q of column c
  auto load_a = [&](int k, int j, T(&v)[4]) {
    const auto p = reinterpret_cast<const __attribute__((address_space(1))) zv*>(as_global(lt + tile_at(k, j)));
#pragma unroll
    for (int e = 0; e < 4 / kOV<T>; ++e) {
      const zv x = p[(4 / kOV<T>) * (4 * c + g) + e];
#pragma unroll
      for (int u = 0; u < kOV<T>; ++u) v[kOV<T> * e + u] = x[u];
    }
  };
  // A operand of -L_kk^{-T}: rows row(g, q) of column c
  auto load_d = [&](int k, T(&v)[4]) {
    const auto p = as_global(lt + tile_at(k, k));
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = p[16 * c + MF<T>::row(g, q)];
  };
#pragma unroll 1
  for (int c0 = 0; c0 < ncol; c0 += kCB * kTile) {
    const int ncb = min(kCB, (ncol - c0 + kTile - 1) / kTile);
    acc_t R[NS][kCB];
    T a0[NS][4], a1[NS][4], dv[4] = {T(0), T(0), T(0), T(0)};
#pragma unroll
    for (int i = 0; i < NS; ++i) {
#pragma unroll
      for (int b = 0; b < kCB; ++b)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int r = kTile * (wave + NW * i) + MF<T>::row(g, t), col = c0 + kTile * b + c;
          T v = T(0);
          if (r < nA) {
            if (col < 2) v = (r < mi) == (col == 0) ? yv[r] : T(0);
            else if (r == mi + col - 2) v = T(1);
          }
          R[i][b][t] = v;
        }
#pragma unroll
      for (int q = 0; q < 4; ++q) a0[i][q] = a1[i][q] = T(0);
    }
    // row k, x -> -X_k = -L_kk^{-T} x in LDS
    auto solve = [&](int k, const acc_t(&x)[kCB]) {
      T* xk = xs + (k & 1) * (kCB * kXT<T>);
      acc_t o[kCB];
#pragma unroll
      for (int b = 0; b < kCB; ++b) o[b] = acc_t{T(0), T(0), T(0), T(0)};
      if (ncb > 1) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int b = 0; b < kCB; ++b) o[b] = MF<T>::mma(dv[q], x[b][q], o[b]);
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) o[0] = MF<T>::mma(dv[q], x[0][q], o[0]);
      }
#pragma unroll
      for (int b = 0; b < kCB; ++b)
#pragma unroll
        for (int t = 0; t < 4; ++t) xk[b * kXT<T> + c * LD + MF<T>::row(g, t)] = o[b][t];
    };
    // X_k to memory: 16 rows of four columns per group of columns, groups dealt to the waves
    auto write = [&](int k) {
      const T* xk = xs + (k & 1) * (kCB * kXT<T>);
      const int r = kTile * k + c;
#pragma unroll
      for (int f = 0; f < 4 * kCB; f += NW) {
        const int q = f + wave, col = c0 + 4 * q + g;  // columns 4 q .. 4 q + 3 of the chunk
        if (q >= 4 * kCB) continue;
        const T v = -xk[(q >> 2) * kXT<T> + (4 * (q & 3) + g) * LD + c];
        if (col < ncol && r < nA) ((__attribute__((address_space(1))) T*)out)[(int64_t)col * nA + r] = v;
      }
    };
    // Step k, k - 1 = NW i0 + w: `a` holds this wave's tiles of row k; those of row k - 1
    // are requested into `an` as a whole, so that they are waited for once, a step later.
    auto step = [&](auto i0c, int w, T(&a)[NS][4], T(&an)[NS][4]) {
      constexpr int i0 = decltype(i0c)::value;
      const int k = NW * i0 + w + 1;
      if (k > nt - 1) return;
      const bool mine = k > 1 && wave == (k - 2) % NW;
      __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
      T xb[kCB][4];
      const T* xk = xs + (k & 1) * (kCB * kXT<T>);
#pragma unroll
      for (int b = 0; b < kCB; ++b)
#pragma unroll
        for (int e = 0; e < 4 / kOV<T>; ++e) {
          const zv x = *reinterpret_cast<const zv*>(xk + b * kXT<T> + c * LD + 4 * g + kOV<T> * e);
#pragma unroll
          for (int u = 0; u < kOV<T>; ++u) xb[b][kOV<T> * e + u] = x[u];
        }
      auto update = [&](int i) {
        if (ncb > 1) {
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int b = 0; b < kCB; ++b) R[i][b] = MF<T>::mma(a[i][q], xb[b][q], R[i][b]);
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q) R[i][0] = MF<T>::mma(a[i][q], xb[0][q], R[i][0]);
        }
      };
#pragma unroll
      for (int i = 0; i < i0; ++i) load_a(k - 1, wave + NW * i, an[i]);
      if (wave < w) load_a(k - 1, wave + NW * i0, an[i0]);
      if (wave <= w) update(i0);
      if (wave == w) solve(k - 1, R[i0]);
      if (mine) load_d(k - 2, dv);
      write(k);
#pragma unroll
      for (int i = 0; i < i0; ++i) update(i);
      __syncthreads();
    };
    {
      const int k = nt - 1;
      if (wave == k % NW) {
        load_d(k, dv);
#pragma unroll
        for (int i = 0; i < NS; ++i)
          if (i == k / NW) solve(k, R[i]);
      }
#pragma unroll
      for (int i = 0; i < NS; ++i)
        if (wave + NW * i < k) {
          if (k & 1) load_a(k, wave + NW * i, a1[i]);
          else load_a(k, wave + NW * i, a0[i]);
        }
      if (k > 0 && wave == (k - 1) % NW) load_d(k - 1, dv);
    }
    __syncthreads();
    unrolled_down<NS>([&](auto i0) {
#pragma unroll 1
      for (int w = NW - 1; w > 0; w -= 2) {  // (NW is even: k = w + 1 mod 2)
        step(i0, w, a0, a1);
        step(i0, w - 1, a1, a0);
      }
    });
    write(0);
    __syncthreads();
  }
}

// LDS of one workgroup (dynamic; the coordinates come last: vectors of two
// dimensions, NTM 16 points per vector row).
template <typename T, int NTM, int NW, int MODE>
struct RowSmem {
  // L of the row being eliminated, operand tiles; the adjoint solves keep the
  // solutions of two steps here
  static constexpr int kRows = (NTM - 1) * 256, kSol = MODE == kAdjoint ? 2 * kCB * kXT<T> : 0;
  alignas(16) T rowb[kRows > kSol ? kRows : kSol];
  alignas(16) T xop[16 * kDg<T>];   // diagonal tile, then minus the inverse of its factor (operand tile)
  alignas(16) T tb[kTile];          // y_k - sum_j L_kj z_j of that row (vec_at order)
  alignas(16) T zk[kTile];          // z_k (vec_at order)
  T yv[NTM * kTile];                // observations, then z
  T pv[NTM * kTile];                // pivots
  T xi[MODE == kSample ? NTM * kTile : 1];   // innovations of the conditional simulator
  T zs[MODE == kSample ? kTile : 1];         // z_c / sqrt(D_c) of the tile
  T rs2[MODE == kSample ? kTile : 1];        // 1 / D_c
  double isc[kMaxDim];              // exp(-theta_k) of the set being processed
  double tab[ExpTable<double>::n];  // table of the exponential
  int flags[NW];
  int next_item;
  alignas(16) double z[1];
};

// CAP > 0 (large blocks): tile_map.  lt: memory of the tiles of L, `stride`
// elements per workgroup (adjoint solves: all of them, and minus the inverses of the
// diagonal tiles; large blocks: those without a register).
template <typename T, int NTM, int NW, int OCC, RowMode MODE, int CAP>
__global__ __launch_bounds__(NW * 64, OCC) void k_block_rows(const SetDesc* __restrict__ sets,
                                                             const double* __restrict__ theta,
                                                             const WorkItem* __restrict__ items,
                                                             const int* __restrict__ count, double piv_tau,
                                                             int* queue, T* tiles, int64_t stride) {
  constexpr bool SAMPLE = MODE == kSample, ADJ = MODE == kAdjoint;
  constexpr bool kAhead = CAP > 0 && NTM <= 14;  // (longer rows: no registers to spare)
  typedef typename MF<T>::acc acc_t;
  typedef RowSmem<T, NTM, NW, MODE> SM;
  constexpr TileMap<NTM, NW> TM = tile_map<NTM, NW, CAP>();
  constexpr int NS = TM.NS, NR = TM.n > 0 ? TM.n : 1;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  SM& sm = *reinterpret_cast<SM*>(smem_raw);
  double* const z = sm.z;
  T* const lt = tiles + (CAP > 0 || ADJ ? (int64_t)blockIdx.x * stride : 0);
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int total = *count;
  if (tid < ExpTable<double>::n) sm.tab[tid] = ExpTable<double>::entry(tid);
  int isc_set = -1;  // set whose coordinate scales sm.isc holds
  auto take = [&](int cur) -> int {
    if (!queue) return cur + gridDim.x;
    if (tid == 0) sm.next_item = atomicAdd(queue, 1);
    __syncthreads();
    const int v = __builtin_amdgcn_readfirstlane(sm.next_item);  // (uniform, and known to be)
    __syncthreads();
    return v;
  };
  for (int it = !queue ? (int)blockIdx.x : take(0); it < total; it = take(it)) {
    const WorkItem w = items[it];
    const SetDesc S = sets[w.set];
    const int d = __builtin_amdgcn_readfirstlane(S.d), nv = (d + kOV<double> - 1) / kOV<double>;
    const double* th = theta + S.theta_off;
    if (w.set != isc_set) {  // uniform over the workgroup
      if (tid < d) sm.isc[tid] = exp(-th[tid]);
      __syncthreads();
      isc_set = w.set;
    }
    const int b0 = S.bptr[w.block], b1 = S.bptr[w.block + 1];
    const int64_t n0 = S.nptr[w.block], n1 = S.nptr[w.block + 1];
    const int mi = __builtin_amdgcn_readfirstlane((int)(n1 - n0)), bi = __builtin_amdgcn_readfirstlane(b1 - b0);
    const int nA = mi + bi, nt = (nA + kTile - 1) / kTile;
    const double sigma2 = exp(th[d]), tau2 = exp(th[d + 1]);
    const T diag0 = T(sigma2) + T(tau2), tau = T(piv_tau);
    const Cov cov(sigma2, S.two_nu);

    bool bad = false, low = false;
    // gather A = J u B (J first), one point per thread, twelve coordinates in
    // flight at once; padding points are zero.  The contraction works with FP32
    // coordinates in the FP32 path: a block whose squared differences could leave
    // their range (20 (2 10^18)^2 < 2^128) goes to the FP64 pass with both kernels.
    for (int pl = tid; pl < nt * kTile; pl += NW * 64) {
      const bool real = pl < nA;
      const int pos = !real ? b0 : pl < mi ? as_global(S.nidx)[n0 + pl] : b0 + (pl - mi);
      const auto xr = as_global(S.X) + (int64_t)pos * d;
      const double yl = as_global(S.y)[pos];
#pragma unroll 1
      for (int e0 = 0; e0 < d; e0 += 12) {
        double x[12];
#pragma unroll
        for (int i = 0; i < 12; ++i) x[i] = xr[min(e0 + i, d - 1)];
#pragma unroll
        for (int i = 0; i < 12; i += kOV<double>) {
          if (e0 + i >= d) continue;
          typename ZV<double>::v v;
#pragma unroll
          for (int u = 0; u < kOV<double>; ++u)
            v[u] = (real && e0 + i + u < d) ? x[i + u] * sm.isc[min(e0 + i + u, d - 1)] : 0.0;
          if constexpr (ADJ && sizeof(T) == 4) {
#pragma unroll
            for (int u = 0; u < kOV<double>; ++u) low |= !(fabs(v[u]) <= 1e18);
          }
          reinterpret_cast<typename ZV<double>::v*>(z)[NTM * kTile * ((e0 + i) / kOV<double>) + pl] = v;
        }
      }
      sm.yv[pl] = (real && (!SAMPLE || pl < mi)) ? T(yl) : T(0);
      if constexpr (SAMPLE)
        sm.xi[pl] = (real && pl >= mi && S.xi) ? T(as_global(S.xi)[b0 - S.out_off + (pl - mi)]) : T(0);
    }
    int row[NS];  // this wave's tile rows (negative: none)
#pragma unroll
    for (int s = 0; s < NS; ++s) row[s] = nt - 1 - NW * s - deal<NW>(s, wave);
    acc_t R[NR];   // tiles of L and accumulators (tile_map)
    acc_t dacc = {T(0), T(0), T(0), T(0)};  // diagonal tile of this wave's next row (negated)
    constexpr bool LOW = sizeof(T) == 4;
    T alow[LOW ? NS : 1][4];                 // low parts of the accumulators' covariances
    T dlow[LOW && CAP > 0 ? NS : 1][4];      // .. of the diagonal tiles'
    T part[NS];    // sum_j L_ij z_j: this lane's columns of row 16 row[s] + c
    T vpart[NS];   // SAMPLE: sum of L_ij^2 over the block's columns, likewise
#pragma unroll
    for (int i = 0; i < NR; ++i) R[i] = acc_t{T(0), T(0), T(0), T(0)};
#pragma unroll
    for (int s = 0; s < NS; ++s) part[s] = vpart[s] = T(0);
    __syncthreads();
    if constexpr (CAP > 0) {  // diagonal tiles
      const int lane = tid & 63;
#pragma unroll 1
      for (int s0 = 0; s0 < NS; ++s0) {
        int r0 = -1;
#pragma unroll
        for (int s = 0; s < NS; ++s) r0 = s == s0 ? row[s] : r0;
        if (r0 < 0) break;
        double v[1][4];
        const int rr[1] = {r0};
        gen_tiles<T, 1, NTM * kTile, true>(z, sm.tab, nv, lane, r0, rr, nt, nA, cov, tau2, v);
#pragma unroll
        for (int s = 0; s < NS; ++s)
          if (s == s0) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              R[TM.dg[s]][t] = T(v[0][t]);
              if (LOW) dlow[LOW ? s : 0][t] = low_part<T>(v[0][t]);
            }
          }
      }
    }
    // publish row r (this wave's slot s): right-hand side of its forward solve
    // and the tiles j < r
    auto publish = [&](int r, int slot, int lane) {
      const int g = lane >> 4, c = lane & 15;
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        if (s != slot) continue;
        const T t = sm.yv[kTile * r + c] - rows_sum(part[s]);
        if (g == 0) sm.tb[vec_at(c)] = t;
#pragma unroll
        for (int j = 0; j < NTM - 1; ++j)
          if (TM.at[s][j] >= 0 && j < r) {
            const acc_t& G = R[TM.at[s][j] >= 0 ? TM.at[s][j] : 0];
            const T v[4] = {G[0], G[1], G[2], G[3]};
            put_operand<T>(sm.rowb + 256 * j, lane, v);
          }
      }
    };
    // Step -1 only prepares and publishes row 0.
    for (int k = -1; k < nt; ++k) {
      // the lane index passes through an empty asm statement: addresses and
      // comparisons made from it are made again in every step instead of being
      // kept in (and spilled from) registers across the loop
      int lane = tid & 63;
      __asm__ volatile("" : "+v"(lane));
      const int g = lane >> 4, c = lane & 15, al = a_lane<T>(lane);
      int act = 0;       // active slots: rows > k
      int nslot = -1;    // slot of row k + 1
      bool own = false;  // row k is this wave's
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        act += row[s] > k ? 1 : 0;
        nslot = row[s] == k + 1 ? s : nslot;
        own |= row[s] == k && k >= 0;  // (rows below 0 do not exist)
      }
      // (opaque: inside the branches on a column the comparisons with k would
      // be folded to constants and kept for the whole loop)
      nslot = __builtin_amdgcn_readfirstlane(nslot);
      __asm__ volatile("" : "+s"(nslot));
      nslot = __builtin_amdgcn_readfirstlane(nslot);
      act = __builtin_amdgcn_readfirstlane(act);
      // the owner of row k factors tile (k, k)
      if (own) {
        // the serial chain of the block: it wins issue arbitration against the
        // other block's wave on this SIMD
        __builtin_amdgcn_s_setprio(3);
        T a[16], wv[4];
        if constexpr (CAP > 0) {
#pragma unroll
          for (int s = 0; s < NS; ++s)
            if (row[s] == k) {
#pragma unroll
              for (int t = 0; t < 4; ++t) sm.xop[c * kDg<T> + MF<T>::row(g, t)] = R[TM.dg[s]][t] + (LOW ? dlow[LOW ? s : 0][t] : T(0));
            }
        } else {
#pragma unroll
          for (int t = 0; t < 4; ++t) sm.xop[c * kDg<T> + MF<T>::row(g, t)] = dacc[t] + (LOW ? dlow[0][t] : T(0));
        }
        __builtin_amdgcn_wave_barrier();
        typedef typename ZV<T>::v zv;
#pragma unroll
        for (int p = 0; p < 16 / kOV<T>; ++p) {
          const zv x = *reinterpret_cast<const zv*>(sm.xop + c * kDg<T> + kOV<T> * p);
#pragma unroll
          for (int e = 0; e < kOV<T>; ++e) a[kOV<T> * p + e] = x[e];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) wv[q] = (g + 4 * q == c) ? T(1) : T(0);
        __builtin_amdgcn_wave_barrier();
        ldl(a, wv);
        // this row's pivot, a[c] (the tile holds -A_kk: the same multipliers, negated
        // pivots)
        T pv = a[0];
#pragma unroll
        for (int e = 1; e < 16; ++e) pv = c == e ? a[e] : pv;
        pv = -pv;
        const T rs = rsqrt_nr(pv);
        T x[4], t[4];
        get_vec<T>(sm.tb, g, t);
        T zp = T(0);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          x[q] = wv[q] * -rs;
          zp -= x[q] * t[q];
        }
        put_operand<T>(sm.xop, lane, x);  // -L_kk^{-1}
        if constexpr (ADJ) tile_store(lt + tile_at(k, k), lane, x);
        T zr = rows_sum(zp);
        const int R0 = kTile * k + c;
        const bool real = R0 < nA;
        if constexpr (SAMPLE) {
          if (R0 >= mi) zr = sm.xi[R0];
          if (g == 0) {
            sm.zs[c] = zr * rs;
            sm.rs2[c] = rs * rs;
          }
          __builtin_amdgcn_wave_barrier();
          const T u = -sm.tb[vec_at(c)];  // (rows of B have no observation: tb = -sum_j L_kj z_j)
          T ysim = u, vv = T(0);
#pragma unroll
          for (int e = 0; e < 16; ++e)
            if (e <= c) {
              ysim -= a[e] * sm.zs[e];
              if (kTile * k + e >= mi) vv += a[e] * a[e] * sm.rs2[e];
            }
          T vs = T(0);
#pragma unroll
          for (int s = 0; s < NS; ++s)
            if (row[s] == k) vs = rows_sum(vpart[s]);
          if (g == 0 && R0 >= mi && real) {
            S.y_out[b0 - S.out_off + R0 - mi] = (double)ysim;
            if (S.var_out) S.var_out[b0 - S.out_off + R0 - mi] = (double)(vs + vv);
          }
        }
        if (g == 0) {
          sm.zk[vec_at(c)] = zr;
          sm.yv[R0] = zr;
          sm.pv[R0] = pv;
        }
        bad |= !(pv > T(0)) || pv > T(3.0e38);
        low |= pv <= tau * (real ? diag0 : T(1));
        __builtin_amdgcn_s_setprio(0);
      }
      if (k == nt - 1) break;
      // column k: -A_ik = -Sigma_ik + sum_j L_ij L_kj^T; two rows at a time share
      // the reads of tile k's points
      for (int s0 = 0; s0 < (k >= 0 ? act : 0); s0 += 2) {
        int r0 = 0, r1 = 0;
#pragma unroll
        for (int s = 0; s < NS; s += 2)
          if (s == s0) {
            r0 = row[s];
            r1 = row[s + 1 < NS ? s + 1 : s];
          }
        if (s0 + 1 < act) {
          double v[2][4];
          const int rr[2] = {r0, r1};
          gen_tiles<T, 2, NTM * kTile>(z, sm.tab, nv, lane, k, rr, nt, nA, cov, tau2, v);
#pragma unroll
          for (int s = 0; s + 1 < NS; s += 2)
            if (s == s0) {
#pragma unroll
              for (int t = 0; t < 4; ++t) {
                R[TM.acc[s]][t] = T(v[0][t]);
                R[TM.acc[s + 1]][t] = T(v[1][t]);
                if (LOW) {
                  alow[LOW ? s : 0][t] = low_part<T>(v[0][t]);
                  alow[LOW ? s + 1 : 0][t] = low_part<T>(v[1][t]);
                }
              }
            }
        } else {
          double v[1][4];
          const int rr[1] = {r0};
          gen_tiles<T, 1, NTM * kTile>(z, sm.tab, nv, lane, k, rr, nt, nA, cov, tau2, v);
#pragma unroll
          for (int s = 0; s < NS; s += 2)
            if (s == s0) {
#pragma unroll
              for (int t = 0; t < 4; ++t) {
                R[TM.acc[s]][t] = T(v[0][t]);
                if (LOW) alow[LOW ? s : 0][t] = low_part<T>(v[0][t]);
              }
            }
        }
      }
      T v[NS][4];  // large: the next tile in memory of each slot
      if constexpr (CAP > 0) {
#pragma unroll
        for (int s = 0; s < NS; ++s)
          if (s < act && TM.res[s] < k) tile_load(lt + tile_at(row[s], TM.res[s]), lane, v[s]);
      }
      // (kAhead: row k's next tile is read while one is used)
      T ap[kAhead ? 2 : 1][4];
      if constexpr (kAhead) get_operand<T>(sm.rowb, al, ap[0]);
#pragma unroll
      for (int j = 0; j < NTM - 1; ++j) {
        if (j >= k || act == 0) continue;
        if constexpr (kAhead) {
          if (j + 1 < NTM - 1) get_operand<T>(sm.rowb + 256 * (j + 1), al, ap[(j + 1) & 1]);
        } else {
          get_operand<T>(sm.rowb + 256 * j, al, ap[0]);
        }
        T(&a)[4] = ap[kAhead ? j & 1 : 0];
#pragma unroll
        for (int s = 0; s < NS; ++s)
          if (TM.at[s][j] >= 0 && s < act) {
            const acc_t& G = R[TM.at[s][j] >= 0 ? TM.at[s][j] : 0];
#pragma unroll
            for (int q = 0; q < 4; ++q) R[TM.acc[s]] = MF<T>::mma(a[q], G[q], R[TM.acc[s]]);
          }
      }
      T fv[TM.fetch > 0 ? TM.fetch : 1][4];  // large: tiles of row k + 1 in memory, for publish()
      int fj = 0;                            // this wave's first one
      if constexpr (CAP > 0) {
        // the columns in memory, in runs of columns that the same slots have there: a
        // tile's registers take its slot's next tile, requested when it has been used
        unrolled_down<NS>([&](auto a1) {
          constexpr int A = decltype(a1)::value + 1;  // active slots
          if (act != A) return;
          unrolled_down<NS>([&](auto p1) {
            constexpr int P = NS - 1 - decltype(p1)::value;
            constexpr int hi = P + 1 < NS ? TM.res[TM.ord[P + 1]] : NTM;
#pragma unroll 1
            for (int j = TM.res[TM.ord[P]]; j < min(hi, k); ++j) {
              T a[4];
              get_operand<T>(sm.rowb + 256 * j, al, a);
#pragma unroll
              for (int s = 0; s < A; ++s) {
                if (TM.rank[s] > P) continue;
#pragma unroll
                for (int q = 0; q < 4; ++q) R[TM.acc[s]] = MF<T>::mma(a[q], v[s][q], R[TM.acc[s]]);
                tile_load(lt + tile_at(row[s], min(j + 1, k - 1)), lane, v[s]);
              }
            }
          });
        });
        const int sn = (nt - 2 - k) / NW;  // slot of row k + 1
#pragma unroll
        for (int s = 0; s < NS; ++s) fj = s == sn ? TM.res[s] + wave : fj;
#pragma unroll
        for (int f = 0; f < TM.fetch; ++f)
          if (fj + NW * f < k) tile_load(lt + tile_at(k + 1, fj + NW * f), lane, fv[f]);
      }
      // the owner of row k + 1 prepares its diagonal tile: covariance and the
      // columns before k
      if (CAP == 0 && nslot >= 0) {
        double v[1][4];
        const int rr[1] = {k + 1};
        gen_tiles<T, 1, NTM * kTile, true>(z, sm.tab, nv, lane, k + 1, rr, nt, nA, cov, tau2, v);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          dacc[t] = T(v[0][t]);
          if (LOW) dlow[0][t] = low_part<T>(v[0][t]);
        }
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          if (s != nslot) continue;
#pragma unroll
          for (int j = 0; j < NTM - 2; ++j)
            if (TM.at[s][j] >= 0 && j < k) {
              const acc_t& G = R[TM.at[s][j] >= 0 ? TM.at[s][j] : 0];
#pragma unroll
              for (int q = 0; q < 4; ++q) dacc = MF<T>::mma(G[q], G[q], dacc);
            }
        }
      }
      __syncthreads();  // -L_kk^{-1} and z_k published
      if (act > 0 && k >= 0) {
        T xo[4], zv4[4];
        get_operand<T>(sm.xop, al, xo);
        get_vec<T>(sm.zk, g, zv4);
        int at_k[NS];  // tiles (row[s], k) in memory (not to be kept per column: opaque)
        if constexpr (CAP > 0 || ADJ) {
#pragma unroll
          for (int s = 0; s < NS; ++s) {
            at_k[s] = __builtin_amdgcn_readfirstlane(tile_at(row[s], k));
            __asm__ volatile("" : "+s"(at_k[s]));
          }
        }
        // (the register a tile goes to is known inside the branch on its column)
#pragma unroll
        for (int j = 0; j < NTM - 1; ++j) {
          if (j != k) continue;
#pragma unroll
          for (int s = 0; s < NS; ++s) {
            if (j >= NTM - 1 - s * NW || s >= act) continue;
            acc_t o = {T(0), T(0), T(0), T(0)};
#pragma unroll
            for (int q = 0; q < 4; ++q)
              o = MF<T>::mma(xo[q], R[TM.acc[s]][q] + (LOW ? alow[LOW ? s : 0][q] : T(0)), o);
#pragma unroll
            for (int q = 0; q < 4; ++q) part[s] += o[q] * zv4[q];
            if constexpr (SAMPLE) {
#pragma unroll
              for (int q = 0; q < 4; ++q)
                if (kTile * j + g + 4 * q >= mi) vpart[s] += o[q] * o[q];
            }
            if (TM.at[s][j] >= 0) R[TM.at[s][j] >= 0 ? TM.at[s][j] : 0] = o;
            if (ADJ || TM.at[s][j] < 0) tile_store(lt + at_k[s], lane, o);
            if constexpr (CAP > 0) {
#pragma unroll
              for (int q = 0; q < 4; ++q) R[TM.dg[s]] = MF<T>::mma(o[q], o[q], R[TM.dg[s]]);
              if (TM.at[s][j] < 0 && s == nslot) {
                const T v[4] = {o[0], o[1], o[2], o[3]};
                put_operand<T>(sm.rowb + 256 * j, lane, v);
              }
            } else if (s == nslot) {
#pragma unroll
              for (int q = 0; q < 4; ++q) dacc = MF<T>::mma(o[q], o[q], dacc);
            }
          }
        }
      }
      publish(k + 1, nslot, lane);
      if constexpr (CAP > 0) {
#pragma unroll
        for (int f = 0; f < TM.fetch; ++f)
          if (fj + NW * f < k) put_operand<T>(sm.rowb + 256 * (fj + NW * f), lane, fv[f]);
      }
      __syncthreads();  // row k + 1 published
    }
    // block term: z^2 and the logarithms of the block's pivots (one logarithm a
    // lane, of the product of its pivots' mantissas), summed in an order that
    // depends on the block alone
    const int fl = (__any(bad) ? 2 : 0) | (__any(low) ? 1 : 0);
    if ((tid & 63) == 0) sm.flags[wave] = fl;
    __syncthreads();
    if (wave == 0) {
      double mant = 1.0, q = 0.0;
      int expo = 0;
      for (int r = mi + tid; r < nA; r += 64) {
        const double p = (double)sm.pv[r], zr = (double)sm.yv[r];
        mant *= __builtin_amdgcn_frexp_mant(p);
        expo += __builtin_amdgcn_frexp_exp(p);
        q += zr * zr;
      }
      double l = log(mant) + (double)expo * 0.693147180559945309417232121458 + q;
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) l += __shfl_xor(l, o, 64);
      if (tid == 0) {
        int f = 0;
        for (int i = 0; i < NW; ++i) f |= sm.flags[i];
        S.llb[w.block] = (f & 2) ? -__builtin_inf() : -0.5 * (l + (double)bi * kLog2Pi);
        S.flag[w.block] = f;
      }
    }
    if constexpr (ADJ) {
      adjoint_solves<T, NTM, NW>(sm.rowb, sm.yv, lt, tid & 63, wave, nt, mi, nA, bi,
                                 reinterpret_cast<T*>(S.qbuf) + S.qoff[w.block]);
    }
    __syncthreads();
  }
}

// ---- variants -------------------------------------------------------------
// Sorted by tile capacity: waves per workgroup and the waves per SIMD its
// registers are capped for, in FP64, in FP32 and with the FP32 adjoint solves (at 14
// tiles, n = 2e5, m = 200, without them two 1303, three 1103, four 2068 us; with them
// two 1561, three 1532 us; 16 tiles two 382, three 446 us).
// cap64, capa64: tiles of a wave in registers
// (tile_map) in FP64 without and with the adjoint solves, 0: all.  With memory for
// the others (one slot per resident workgroup) nothing is spilled and the diagonal
// tiles need no preparation: of n = 1e6, m = 200 the 15-tile blocks take 2155 us
// instead of 2444 (cap 10: 2242, 12: 2167, 14: 2160, 16: 2155), the 14-tile ones 7820
// instead of 8060 (cap 10: 8005, 12: 7909, 14: 7820, 16: 7880, 18: 8095).  With the
// adjoint solves, n = 2e5: 16-tile variant 668 instead of 747 us, 14-tile 2270 instead
// of 2160.  Three blocks per unit spill in every loop (14 tiles: 9250 us).  (Sweeps
// made before the exponential underflowed to 0, which added up to 1 %.)
struct RowVariant {
  int ntm, nw, occ64, occ32, adj32, cap64, capa64;
};
static constexpr RowVariant kRow[] = {{4, 2, 4, 4, 4, 0, 0},   {8, 4, 3, 4, 4, 0, 0},    {12, 4, 2, 3, 3, 0, 0},
                                      {14, 4, 2, 3, 3, 14, 0}, {16, 4, 2, 2, 2, 14, 14}, {17, 4, 2, 2, 2, 14, 14}};
constexpr int kNumVariants = sizeof(kRow) / sizeof(kRow[0]);


// One launch: `tiles` with `stride` elements per workgroup for the tiles of L, where
// the launch needs them.
template <typename T, int NTM, int NW, int OCC, RowMode MODE, int CAP>
static hipError_t launch_rows(int grid, int dmax, const SetDesc* sets, const double* theta, const WorkItem* items,
                              const int* count, double piv_tau, int* queue, T* tiles, hipStream_t s) {
  typedef RowSmem<T, NTM, NW, MODE> SM;
  if (dmax < 1 || dmax > kMaxDim) return hipErrorInvalidValue;
  const int ld = (dmax + kOV<double> - 1) / kOV<double> * kOV<double>;  // whole vectors
  const size_t lds = offsetof(SM, z) + sizeof(double) * NTM * kTile * ld;
  hipLaunchKernelGGL((k_block_rows<T, NTM, NW, OCC, MODE, CAP>), dim3(grid), dim3(NW * 64), lds, s, sets, theta, items,
                     count, piv_tau, queue, tiles, tile_elems(NTM));
  return hipGetLastError();
}

template <typename T, RowMode MODE>
static hipError_t launch_rows_v(int v, int grid, int dmax, const SetDesc* sets, const double* theta,
                                const WorkItem* items, const int* count, double piv_tau, int* queue, T* tiles,
                                hipStream_t s) {
#define SBV_LAUNCH(V, OCC, CAP)                                                                                  \
  launch_rows<T, kRow[V].ntm, kRow[V].nw, OCC, MODE, CAP>(grid, dmax, sets, theta, items, count, piv_tau, queue, \
                                                          tiles, s)
#define SBV_ROWS(V)                                                                                       \
  case V: {                                                                                               \
    constexpr bool A = MODE == kAdjoint, D = sizeof(T) == 8;                                              \
    constexpr int occ = D ? kRow[V].occ64 : A ? kRow[V].adj32 : kRow[V].occ32;                            \
    constexpr int cap = !D || MODE == kSample ? 0 : A ? kRow[V].capa64 : kRow[V].cap64;                   \
    if constexpr (A) return SBV_LAUNCH(V, occ, cap);                                                      \
    return tiles && cap ? SBV_LAUNCH(V, occ, cap) : SBV_LAUNCH(V, occ, 0);                                \
  }
  switch (v) {
    SBV_ROWS(0) SBV_ROWS(1) SBV_ROWS(2) SBV_ROWS(3) SBV_ROWS(4) SBV_ROWS(5)
  }
#undef SBV_ROWS
#undef SBV_LAUNCH
  return hipErrorInvalidValue;
}

}  // namespace sbv
