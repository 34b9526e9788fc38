// Axis-pass kernels: double forward, lengths of part 3.
#include "kernels_pass.hpp"

namespace fftb {
FFTB_PASS_INST(, -1, double, 3)
}  // namespace fftb
