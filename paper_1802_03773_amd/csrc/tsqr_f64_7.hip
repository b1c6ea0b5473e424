// Instantiation of the float64 tall-skinny QR for 7 column block(s) of 16.
#include "tsqr_f64.hpp"

namespace qrk {
QRK_TSQR64_INST(7)
}  // namespace qrk
