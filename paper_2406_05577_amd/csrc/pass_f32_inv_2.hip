// Axis-pass kernels: complex64, inverse, lengths of part 2.
#include "kernels_pass.hpp"

namespace fftb {
FFTB_PASS_INST(, +1, float, 1, 2)
}  // namespace fftb
