// Launch of the pipelined dense-part merge tree (see tsqr_tree.hpp), one instantiation per
// column-block count 1 .. 8.
#include "qrk_launch.hpp"
#include "tsqr_tree.hpp"

namespace qrk {

hipError_t launch_tsqr_tree(int ncb, const ProbDesc* probs, const TreeNodes& tn, float* slots, int* flags, float* RB,
                            int* status, const QStore& qs, hipStream_t st) {
  if (tn.count < 1) return hipSuccess;
  switch (ncb) {
#define QRK_TREE(N)                                                                                          \
  case N: {                                                                                                  \
    const int wpg = tree_waves(N, qs.qn != nullptr);                                                         \
    const dim3 grid((unsigned)((tn.count + wpg - 1) / wpg)), blk(64 * wpg);                                    \
    if (qs.qn)                                                                                               \
      hipLaunchKernelGGL((k_tsqr_tree_keep<N>), grid, blk, 0, st, probs, tn, slots, flags, RB, status, qs);     \
    else                                                                                                     \
      hipLaunchKernelGGL((k_tsqr_tree<N>), grid, blk, 0, st, probs, tn, slots, flags, RB, status);              \
    break;                                                                                                   \
  }
    QRK_TREE(1) QRK_TREE(2) QRK_TREE(3) QRK_TREE(4) QRK_TREE(5) QRK_TREE(6) QRK_TREE(7) QRK_TREE(8)
#undef QRK_TREE
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace qrk
