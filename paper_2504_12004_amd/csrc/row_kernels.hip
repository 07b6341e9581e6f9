// Launchers of the block kernel: log-likelihood terms and conditional simulation.
#include "row_block.h"

namespace sbv {

int n_variants() { return kNumVariants; }
Variant variant(int v) { return Variant{kRow[v].ntm, kRow[v].nw}; }
int waves_per_cu(int prec, int v) { return 4 * (prec == 0 ? kRow[v].occ64 : kRow[v].occ32); }
int tile_slots(int prec, int v) { return prec == 0 && kRow[v].cap64 ? kUnits * (4 * kRow[v].occ64 / kRow[v].nw) : 0; }
int variant_for(int nA) {
  for (int v = 0; v < kNumVariants; ++v)
    if (nA <= kRow[v].ntm * kTile) return v;
  return -1;
}

hipError_t launch_loglik(int prec, int v, int grid, int dmax, const SetDesc* sets, const double* theta,
                         const WorkItem* items, const int* count, double piv_tau, hipStream_t s, int* queue,
                         double* tiles) {
  if (grid <= 0) return hipSuccess;
  if (prec == 0)
    return launch_rows_v<double, kValue>(v, grid, dmax, sets, theta, items, count, piv_tau, queue, tiles, s);
  return launch_rows_v<float, kValue>(v, grid, dmax, sets, theta, items, count, piv_tau, queue, nullptr, s);
}

hipError_t launch_sample(int v, int grid, int dmax, const SetDesc* sets, const double* theta, const WorkItem* items,
                         const int* count, hipStream_t s) {
  if (grid <= 0) return hipSuccess;
  return launch_rows_v<double, kSample>(v, grid, dmax, sets, theta, items, count, 0.0, nullptr, nullptr, s);
}

}  // namespace sbv
