// Plane kernels: complex128.
#include "kernels_plane.hpp"

namespace fftb {
template hipError_t plane_launch<double, 1>(PassMode, const PlaneArgs&, int, size_t, hipStream_t, bool);
}  // namespace fftb
