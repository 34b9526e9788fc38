// Axis-pass kernels: double forward, lengths of part 0.
#include "kernels_pass.hpp"

namespace fftb {
FFTB_PASS_INST(, -1, double, 0)
}  // namespace fftb
