// Plane kernels: complex64, two bands per lane.
#include "kernels_plane.hpp"

namespace fftb {
template hipError_t plane_launch<float, 2>(PassMode, const PlaneArgs&, int, size_t, hipStream_t, bool);
}  // namespace fftb
