// Instantiation of the float64 tall-skinny QR for 4 column block(s) of 16.
#include "tsqr_f64.hpp"

namespace qrk {
QRK_TSQR64_INST(4)
}  // namespace qrk
