// Axis-pass kernels: complex64, two bands per lane, x pass of the potential step, lengths of part 2.
#include "kernels_pass.hpp"

namespace fftb {
FFTB_PASS_INST(, 2, float, 2, 2)
}  // namespace fftb
