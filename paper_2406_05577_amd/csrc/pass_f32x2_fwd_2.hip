// Axis-pass kernels: complex64, two bands per lane, forward, lengths of part 2.
#include "kernels_pass.hpp"

namespace fftb {
FFTB_PASS_INST(, -1, float, 2, 2)
}  // namespace fftb
