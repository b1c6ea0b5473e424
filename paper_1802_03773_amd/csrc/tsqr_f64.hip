// Dispatch of the float64 tall-skinny QR (tsqr_f64.hpp): per column-block count present, one
// launch of all its problems' leaves and one of all their merge nodes.
#include "qrk_launch.hpp"
#include "tsqr_f64.hpp"

namespace qrk {

int tsqr64_slot_doubles(int L) {
  const int ncb = (L + 15) / 16;
  return ncb * (ncb + 1) / 2 * 256;
}
int tsqr64_tile_rows(int ncb) { return leaf_tile_rows_f64(ncb); }

#define QRK_T64_EACH(X) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8)

hipError_t launch_tsqr64_leaves(int ncb, int leaf_begin, int count, const int32_t* leaf_prob, const int32_t* leaf_idx,
                                const ProbDesc* probs, int n, const double* Red, const double* d, const double* lam,
                                double* slots, double* RB, hipStream_t st) {
  if (count < 1) return hipSuccess;
  switch (ncb) {
#define QRK_T64(N) \
  case N:          \
    return launch_tsqr64_leaf_n<N>(leaf_begin, count, leaf_prob, leaf_idx, probs, n, Red, d, lam, slots, RB, st);
    QRK_T64_EACH(QRK_T64)
#undef QRK_T64
    default:
      return hipErrorInvalidValue;
  }
}

hipError_t launch_tsqr64_tree(int ncb, int node_begin, int count, const int32_t* node_prob, const int32_t* node_idx,
                              const int32_t* node_l, const int32_t* node_r, const ProbDesc* probs, double* slots,
                              int* flags, int* ticket, double* RB, int* status, hipStream_t st) {
  if (count < 1) return hipSuccess;
  switch (ncb) {
#define QRK_T64(N)                                                                                              \
  case N:                                                                                                       \
    return launch_tsqr64_tree_n<N>(node_begin, count, node_prob, node_idx, node_l, node_r, probs, slots, flags, \
                                   ticket, RB, status, st);
    QRK_T64_EACH(QRK_T64)
#undef QRK_T64
    default:
      return hipErrorInvalidValue;
  }
}

}  // namespace qrk
