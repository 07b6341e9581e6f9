// Internal types shared by the HIP kernels and the C-ABI layer of libsbv.so.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>
#include <vector>

namespace sbv {

// Tile edge of every block factorisation (the 16x16 MFMA output tile).
constexpr int kTile = 16;
constexpr int kUnits = 256;  // compute units of the device
// Largest input dimension supported by the fused kernels.
constexpr int kMaxDim = 20;

// One dataset as the kernels see it: points in block-rank order.
struct SetDesc {
  const double* X;        // n x d, row-major, rank order
  const double* y;        // n, rank order
  const int32_t* bptr;    // K+1 block offsets into the ordered points
  const int64_t* nptr;    // K+1 offsets into nidx
  const int32_t* nidx;    // conditioning points as ordered positions
  double* llb;            // K per-block terms (output)
  int32_t* flag;          // K per-block status (output): bit0 fp32 pivot flag, bit1 not PD
  double* gradb;          // K x (d+2) per-block gradient terms (output, gradient kernels)
  double* qbuf;           // adjoint buffer: per block e, g, Q (elements of the kernel precision)
  const int64_t* qoff;    // K offsets into qbuf, in elements of the kernel precision
  const double* xi;       // n innovations, rank order (conditional simulation only; null: all 0)
  double* y_out;          // simulated observations, rank order (conditional simulation only)
  double* var_out;        // conditional variances of the block points (prediction only; may be null)
  int32_t d;
  int32_t two_nu;
  int32_t theta_off;      // offset of this set's d+2 parameters in the theta buffer
  int32_t K;
  int32_t out_off;        // xi, y_out and var_out are indexed by (ordered position - out_off)
};

// One unit of work: block `block` of set `set`.
struct WorkItem {
  int32_t set;
  int32_t block;
};

// Kernel variant: capacity of ntm 16-row tiles per side, nw waves.
struct Variant {
  int ntm;
  int nw;
};

// Blocks whose joint size exceeds the largest variant's capacity (kLargeNTM tiles)
// run with part of the factor in memory, up to 512 points.
constexpr int kLargeNTM = 17;
constexpr int kMaxPrefix = 15;  // tiles beyond kLargeNTM
// Elements of the tiles of L of a block of ntm tile rows (kept in memory by the
// adjoint solves and, those without a register, by large blocks).
constexpr int64_t tile_elems(int ntm) { return (int64_t)256 * ntm * (ntm + 1) / 2; }

// Tile rows of a large block beyond kLargeNTM, or -1 when it is not one: it fits a
// register variant, exceeds 512 points, or has fewer conditioning points than those
// rows (a handle refuses such a block).
inline int large_prefix(int nA, int mi) {
  const int nt = (nA + kTile - 1) / kTile;
  const int p = nt - kLargeNTM;
  if (p < 1 || p > kMaxPrefix || kTile * p > mi) return -1;
  return p;
}

// Launchers (row_kernels.hip, row_adjoint_kernels.hip, row_large_kernels.hip,
// contract_kernels.hip, loglik_kernels.hip).  `count` is a device int; the kernel
// loops over items[blockIdx.x + k*gridDim.x] while the index is below *count.
// dmax is the largest input dimension among the sets (it sizes the LDS).  With
// `queue` set, workgroups take their items from that device counter instead (one
// atomic increment per item, starting at 0), so that one persistent launch can
// serve every item of a list whatever the number of resident workgroups.  Variants
// with tile_slots > 0 run faster with memory for a part of the factor: tiles,
// tile_elems(ntm) doubles for each of at most tile_slots workgroups.
hipError_t launch_loglik(int prec, int variant, int grid, int dmax, const SetDesc* sets, const double* theta,
                         const WorkItem* items, const int* count, double piv_tau, hipStream_t s,
                         int* queue = nullptr, double* tiles = nullptr);
int tile_slots(int prec, int variant);
// Factorisation with the adjoint solves (gradient): as launch_loglik, and leaves
// e, g and Q in the sets' adjoint buffers.  tiles: tile_elems(ntm) elements of the
// kernel precision per workgroup; adjoint_slots is the number of workgroups that
// are resident at once.
hipError_t launch_loglik_adjoint(int prec, int variant, int grid, int dmax, const SetDesc* sets, const double* theta,
                                 const WorkItem* items, const int* count, double piv_tau, void* tiles, hipStream_t s);
int adjoint_slots(int prec, int variant);
// Large blocks (joint sizes above the variants', up to max_joint), with the adjoint
// solves when asked for.  tiles: tile_elems(large_ntm(max_joint)) elements of the
// kernel precision per workgroup.
hipError_t launch_large(int prec, bool adjoint, int max_joint, int grid, int dmax, const SetDesc* sets,
                        const double* theta, const WorkItem* items, const int* count, double piv_tau, void* tiles,
                        hipStream_t s);
int large_ntm(int nA);  // tile rows of the smallest large variant holding nA, or -1
int large_slots(int prec, bool adjoint);  // workgroups of it that are resident at once
// Gradient contraction of blocks with joint sizes up to max_joint.
hipError_t launch_contract(int prec, int max_joint, int grid, int dmax, const SetDesc* sets, const double* theta,
                           const WorkItem* items, const int* count, hipStream_t s);
hipError_t launch_sample(int variant, int grid, int dmax, const SetDesc* sets, const double* theta,
                         const WorkItem* items, const int* count, hipStream_t s);
// bad (n_sets, may be null): the not-positive-definite flags written by
// launch_reduce; a flagged set's gradient is NaN.
hipError_t launch_reduce_grad(const SetDesc* sets, int n_sets, int dmax, double* out, const int* bad, hipStream_t s);
int n_variants();
Variant variant(int v);
int waves_per_cu(int prec, int variant);  // waves of a variant that fit a compute unit's registers
int variant_for(int nA);  // smallest variant holding a joint size nA, or -1

// Lists of blocks, one per register variant: a list with fewer than kMinBucket
// blocks joins the next larger variant's list, if there is one.  A launch of so
// few blocks leaves compute units idle and lasts as long as one block (15-60 us);
// in a longer list, longest blocks first, they fill the last wave of blocks instead
// (n = 2e5, m = 200: three launches of 87 us together become none, the long list's
// launch does not get longer).  A block's arithmetic does not depend on the variant.
constexpr size_t kMinBucket = 256;
template <typename List>
void merge_small(std::vector<List>& per) {
  for (int v = 0; v + 1 < n_variants(); ++v) {
    if (per[v].empty() || per[v].size() >= kMinBucket) continue;
    int u = v + 1;
    while (u < n_variants() && per[u].empty()) ++u;
    if (u == n_variants()) continue;
    per[u].insert(per[u].end(), per[v].begin(), per[v].end());
    per[v].clear();
  }
}
hipError_t launch_reduce(const SetDesc* sets, int n_sets, double* out, int* bad, hipStream_t s);
hipError_t launch_flag_compact(const SetDesc* sets, const WorkItem* items, const int* count,
                               WorkItem* out_items, int* out_count, hipStream_t s);
hipError_t launch_zero_int(int* p, int n, hipStream_t s);
int max_grid(int variant);  // workgroups of a launch whose number of blocks only the device knows

}  // namespace sbv

namespace sbv {

// Read-only view of a handle for entry points outside the evaluation plans:
// its device arrays and the work lists made when the handle was created (one
// size bucket per register variant, longest joint size first, items of set 0,
// all in one device array with one device count per bucket).
struct HandleView {
  const double* X;
  const double* y;
  const int32_t* bptr;
  const int64_t* nptr;
  const int32_t* nidx;
  int32_t d;
  int64_t K;
  int32_t max_joint;
  bool has_large;                 // some block needs the large-joint-set path
  int n_buckets;
  const int* bucket_variant;      // host, n_buckets
  const int* bucket_off;          // host, n_buckets: offset into items
  const int* bucket_count;        // host, n_buckets
  const WorkItem* items;          // device, K items grouped by bucket
  const int* dcount;              // device, n_buckets counts
  const int64_t* block_pts_host;  // host, n: original id of each ordered position
  int64_t n;
};

// Neighbour search of the builder (build_kernels.hip): brute force over the
// points of earlier blocks for queries 0..K-1 or the ascending ranks in qlist,
// and the two steps of the filtered search (coarse candidate blocks, fine
// candidate points with its exactness status).
hipError_t launch_knn(const double* Z, int d, const double* cen, const int32_t* bptr, int K, int m,
                      const int64_t* nn_ptr, int32_t* nn_pos, hipStream_t s, const int32_t* qlist = nullptr,
                      int nq = 0);
hipError_t launch_knn_coarse(const double* cen, const double* rad, int d, const int32_t* qlist, int nq,
                             const double* lam, int cap, int32_t* cand, int32_t* ccount, hipStream_t s);
hipError_t launch_knn_fine(const double* Z, int d, const double* cen, const int32_t* bptr, const int32_t* qlist,
                           int nq, const double* lam, int cap, const int32_t* cand, const int32_t* ccount,
                           const int64_t* nn_ptr, int32_t* nn_pos, int32_t* status, hipStream_t s);
int knn_max_m();

// Dense covariance matrix between two point lists (device buffers; theta on
// the device, d + 2 log-parameters).
hipError_t launch_cov_matrix(const double* Xa, int64_t na, const double* Xb, int64_t nb, int d, const double* theta,
                             int two_nu, int same, double* out, hipStream_t s);

// Pivot threshold of the FP32 path (a block whose FP32 pivot falls to or
// below this fraction of its original diagonal is recomputed in FP64).
double fp32_pivot_tau();

// Summaries of n_draws draws mean_j + sqrt(var_j) xi[t * n + j] per point j:
// stats[j] sample mean, stats[n + j] sample variance (divisor n_draws - 1),
// stats[2n + j] / stats[3n + j] the 95 % interval mean -/+ z sd.
hipError_t launch_pred_draws(const double* mean, const double* var, int64_t n, const double* xi, int n_draws,
                             double* stats, hipStream_t s);

hipError_t launch_gather_y(const double* y_ord, const int32_t* pos_of, double* y, int64_t n, hipStream_t s);
hipError_t launch_scatter_y(const double* y, const int32_t* pos_of, double* y_ord, int64_t n,
                            hipStream_t s);
}  // namespace sbv
