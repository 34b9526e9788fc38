// Axis-pass kernels: double inverse, lengths of part 2.
#include "kernels_pass.hpp"

namespace fftb {
FFTB_PASS_INST(, +1, double, 2)
}  // namespace fftb
