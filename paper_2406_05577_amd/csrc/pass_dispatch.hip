// Axis-pass and plane-kernel dispatch: the launchers the host calls. The kernels
// are instantiated in the pass_*.hip and plane_*.hip translation units.
#include "kernels_plane.hpp"

namespace fftb {

#define FFTB_PASS_DECL(S, T, V) \
  FFTB_PASS_INST(extern, S, T, V, 0) FFTB_PASS_INST(extern, S, T, V, 1) \
  FFTB_PASS_INST(extern, S, T, V, 2) FFTB_PASS_INST(extern, S, T, V, 3)
FFTB_PASS_DECL(+1, float, 1)
FFTB_PASS_DECL(-1, float, 1)
FFTB_PASS_DECL(+1, float, 2)
FFTB_PASS_DECL(-1, float, 2)
FFTB_PASS_DECL(+1, double, 1)
FFTB_PASS_DECL(-1, double, 1)
FFTB_PASS_DECL(+2, float, 1)
FFTB_PASS_DECL(+2, float, 2)
FFTB_PASS_DECL(+2, double, 1)

extern template hipError_t plane_launch<float, 1>(PassMode, const PlaneArgs&, int, size_t, hipStream_t, bool);
extern template hipError_t plane_launch<float, 2>(PassMode, const PlaneArgs&, int, size_t, hipStream_t, bool);
extern template hipError_t plane_launch<double, 1>(PassMode, const PlaneArgs&, int, size_t, hipStream_t, bool);

namespace {
template <int S, typename T, int V>
hipError_t any_part(int n, const PassArgs& a, int threads, size_t lds, hipStream_t st, bool attr) {
  bool found = false;
  hipError_t e = pass_part<S, T, V, 0>(n, a, threads, lds, st, attr, &found);
  if (!found) e = pass_part<S, T, V, 1>(n, a, threads, lds, st, attr, &found);
  if (!found) e = pass_part<S, T, V, 2>(n, a, threads, lds, st, attr, &found);
  if (!found) e = pass_part<S, T, V, 3>(n, a, threads, lds, st, attr, &found);
  return e;
}
template <int S>
hipError_t dispatch(PassElem el, int n, const PassArgs& a, int threads, size_t lds, hipStream_t st, bool attr) {
  switch (el) {
    case kElemC128: return any_part<S, double, 1>(n, a, threads, lds, st, attr);
    case kElemC64x2: return any_part<S, float, 2>(n, a, threads, lds, st, attr);
    default: return any_part<S, float, 1>(n, a, threads, lds, st, attr);
  }
}
}  // namespace

hipError_t launch_pass(PassMode mode, PassElem el, int n, const PassArgs& a, int threads, size_t lds,
                       hipStream_t st) {
  return mode == kPassInverse   ? dispatch<+1>(el, n, a, threads, lds, st, false)
         : mode == kPassForward ? dispatch<-1>(el, n, a, threads, lds, st, false)
                                : dispatch<+2>(el, n, a, threads, lds, st, false);
}

// Allow the kernels of length n `lds` bytes of dynamic LDS.
hipError_t prepare_pass(PassMode mode, PassElem el, int n, size_t lds) {
  PassArgs a{};
  return mode == kPassInverse   ? dispatch<+1>(el, n, a, 0, lds, nullptr, true)
         : mode == kPassForward ? dispatch<-1>(el, n, a, 0, lds, nullptr, true)
                                : dispatch<+2>(el, n, a, 0, lds, nullptr, true);
}

namespace {
hipError_t plane(PassMode mode, PassElem el, const PlaneArgs& a, int threads, size_t lds, hipStream_t st,
                 bool attr) {
  switch (el) {
    case kElemC128: return plane_launch<double, 1>(mode, a, threads, lds, st, attr);
    case kElemC64x2: return plane_launch<float, 2>(mode, a, threads, lds, st, attr);
    default: return plane_launch<float, 1>(mode, a, threads, lds, st, attr);
  }
}
}  // namespace

hipError_t launch_plane(PassMode mode, PassElem el, const PlaneArgs& a, int threads, size_t lds, hipStream_t st) {
  return plane(mode, el, a, threads, lds, st, false);
}

// Allow the plane kernels `lds` bytes of dynamic LDS.
hipError_t prepare_plane(PassMode mode, PassElem el, size_t lds) {
  return plane(mode, el, PlaneArgs{}, 0, lds, nullptr, true);
}

}  // namespace fftb
