// Axis-pass kernels: complex128, forward, lengths of part 1.
#include "kernels_pass.hpp"

namespace fftb {
FFTB_PASS_INST(, -1, double, 1, 1)
}  // namespace fftb
