// Axis-pass kernels: complex64, x pass of the potential step, lengths of part 1.
#include "kernels_pass.hpp"

namespace fftb {
FFTB_PASS_INST(, 2, float, 1, 1)
}  // namespace fftb
