// Axis-pass kernels: complex64, two bands per lane, inverse, lengths of part 0.
#include "kernels_pass.hpp"

namespace fftb {
FFTB_PASS_INST(, +1, float, 2, 0)
}  // namespace fftb
