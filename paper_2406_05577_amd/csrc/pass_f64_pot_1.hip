// Axis-pass kernels: complex128, x pass of the potential step, lengths of part 1.
#include "kernels_pass.hpp"

namespace fftb {
FFTB_PASS_INST(, 2, double, 1, 1)
}  // namespace fftb
