// Instantiation of the lane-ring Givens QR for double, band widths 1 .. 15.
#include "banded_s.hpp"

namespace qrk {

QRK_BS_INST(double, 0, 1, 16)

}  // namespace qrk
