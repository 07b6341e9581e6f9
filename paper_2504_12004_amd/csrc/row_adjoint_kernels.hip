// Launchers of the block kernel with the adjoint solves.
#include "row_block.h"

namespace sbv {

int adjoint_slots(int prec, int v) { return kUnits * (4 * (prec == 0 ? kRow[v].occ64 : kRow[v].adj32) / kRow[v].nw); }

hipError_t launch_loglik_adjoint(int prec, int v, int grid, int dmax, const SetDesc* sets, const double* theta,
                                 const WorkItem* items, const int* count, double piv_tau, void* tiles, hipStream_t s) {
  if (grid <= 0) return hipSuccess;
  if (prec == 0)
    return launch_rows_v<double, kAdjoint>(v, grid, dmax, sets, theta, items, count, piv_tau, nullptr, (double*)tiles,
                                           s);
  return launch_rows_v<float, kAdjoint>(v, grid, dmax, sets, theta, items, count, piv_tau, nullptr, (float*)tiles, s);
}

}  // namespace sbv
