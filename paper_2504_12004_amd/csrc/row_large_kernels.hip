// Launchers of the block kernel for large blocks.
#include "row_block.h"

namespace sbv {

// Waves per workgroup, waves per SIMD and tiles of a wave in registers.  A wave's
// share of a block of 28 tile rows is 47 tiles; the ones that are not kept are
// read again from memory for every later column.  Measured at n = 1e5, m = 400 (FP64;
// kernel time, us), tiles kept in registers / waves per SIMD:
//   8 waves, 2 per SIMD:  8: 6118  12: 5506  14: 5359  16: 5287  18: 5767  22: 5914
//   12 waves, 3 per SIMD: 8: 6425  10: 6100      16 waves, 4 per SIMD: 4: 6809  6: 6596
// Above 16 the compiler spills what is needed in every step.  FP32 (its covariances
// are made in FP64 too): 3000 blocks, m = 400, 2 per SIMD 20: 2925  24: 2879  28: 2792,
// 4 per SIMD (two blocks per unit) 12: 4027; with the adjoint solves (2500 blocks) 2
// per SIMD 20: 2151  24: 2176  32: 2214.
struct LargeVariant {
  int nw, occ, cap;
};
constexpr LargeVariant kBig64{8, 2, 16}, kBig32{8, 2, 28}, kBig32Adj{8, 2, 20};
constexpr int kBigNTM[] = {24, 28, 32};
template <typename T, RowMode MODE>
constexpr LargeVariant kBig = sizeof(T) == 8 ? kBig64 : MODE == kAdjoint ? kBig32Adj : kBig32;

int large_ntm(int nA) {
  for (int ntm : kBigNTM)
    if (nA <= ntm * kTile) return ntm;
  return -1;
}
int large_slots(int prec, bool adjoint) {
  const LargeVariant v = prec == 0 ? kBig64 : adjoint ? kBig32Adj : kBig32;
  return kUnits * (4 * v.occ / v.nw);
}

template <typename T, RowMode MODE>
static hipError_t launch_big(int ntm, int grid, int dmax, const SetDesc* sets, const double* theta,
                             const WorkItem* items, const int* count, double piv_tau, T* tiles, hipStream_t s) {
  constexpr LargeVariant B = kBig<T, MODE>;
#define SBV_BIG(V)                                                                                               \
  if (ntm == kBigNTM[V])                                                                                         \
    return launch_rows<T, kBigNTM[V], B.nw, B.occ, MODE, B.cap>(grid, dmax, sets, theta, items, count, piv_tau, \
                                                                nullptr, tiles, s);
  SBV_BIG(0) SBV_BIG(1) SBV_BIG(2)
#undef SBV_BIG
  return hipErrorInvalidValue;
}

hipError_t launch_large(int prec, bool adjoint, int max_joint, int grid, int dmax, const SetDesc* sets,
                        const double* theta, const WorkItem* items, const int* count, double piv_tau, void* tiles,
                        hipStream_t s) {
  if (grid <= 0) return hipSuccess;
  const int ntm = large_ntm(max_joint);
  if (prec == 0)
    return adjoint ? launch_big<double, kAdjoint>(ntm, grid, dmax, sets, theta, items, count, piv_tau, (double*)tiles, s)
                   : launch_big<double, kValue>(ntm, grid, dmax, sets, theta, items, count, piv_tau, (double*)tiles, s);
  return adjoint ? launch_big<float, kAdjoint>(ntm, grid, dmax, sets, theta, items, count, piv_tau, (float*)tiles, s)
                 : launch_big<float, kValue>(ntm, grid, dmax, sets, theta, items, count, piv_tau, (float*)tiles, s);
}

}  // namespace sbv
