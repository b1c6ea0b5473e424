// Instantiation of the lane-ring Givens QR for float, band widths 1 .. 15.
#include "banded_s.hpp"

namespace qrk {

QRK_BS_INST(float, 0, 1, 16)

}  // namespace qrk
