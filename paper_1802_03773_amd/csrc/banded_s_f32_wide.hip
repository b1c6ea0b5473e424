// Instantiation of the lane-ring Givens QR for float, band widths 16 .. 31, and of the wide-band sweeps.
#include "banded_s.hpp"

namespace qrk {

QRK_BS_INST(float, 1, 16, 32)

template <>
hipError_t launch_bsweep_x<float>(int kind, int P, int64_t N, int w, const float* Rb, const double* binv, const float* rhsT,
                              const double* rhsD, double* out, int* status, hipStream_t st) {
  return launch_bsweep_x_t<float>(kind, P, N, w, Rb, binv, rhsT, rhsD, out, status, st);
}

}  // namespace qrk
