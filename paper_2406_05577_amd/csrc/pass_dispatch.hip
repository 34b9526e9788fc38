// Axis-pass dispatch: the launchers the host calls. The kernels are
// instantiated in the pass_*.hip translation units.
#include "kernels_pass.hpp"

namespace fftb {

#define FFTB_PASS_DECL(S, T) \
  FFTB_PASS_INST(extern, S, T, 0) FFTB_PASS_INST(extern, S, T, 1) \
  FFTB_PASS_INST(extern, S, T, 2) FFTB_PASS_INST(extern, S, T, 3)
FFTB_PASS_DECL(+1, float)
FFTB_PASS_DECL(-1, float)
FFTB_PASS_DECL(+1, double)
FFTB_PASS_DECL(-1, double)

namespace {
template <int S, typename T>
hipError_t any_part(int n, const PassArgs& a, int threads, size_t lds, hipStream_t st, bool attr) {
  bool found = false;
  hipError_t e = pass_part<S, T, 0>(n, a, threads, lds, st, attr, &found);
  if (!found) e = pass_part<S, T, 1>(n, a, threads, lds, st, attr, &found);
  if (!found) e = pass_part<S, T, 2>(n, a, threads, lds, st, attr, &found);
  if (!found) e = pass_part<S, T, 3>(n, a, threads, lds, st, attr, &found);
  return e;
}
hipError_t dispatch(bool inverse, bool fp64, int n, const PassArgs& a, int threads, size_t lds,
                    hipStream_t st, bool attr) {
  if (fp64)
    return inverse ? any_part<+1, double>(n, a, threads, lds, st, attr)
                   : any_part<-1, double>(n, a, threads, lds, st, attr);
  return inverse ? any_part<+1, float>(n, a, threads, lds, st, attr)
                 : any_part<-1, float>(n, a, threads, lds, st, attr);
}
}  // namespace

hipError_t launch_pass(bool inverse, bool fp64, int n, const PassArgs& a, int threads, size_t lds,
                       hipStream_t st) {
  return dispatch(inverse, fp64, n, a, threads, lds, st, false);
}

// Allow the kernels of length n `lds` bytes of dynamic LDS.
hipError_t prepare_pass(bool inverse, bool fp64, int n, size_t lds) {
  PassArgs a{};
  return dispatch(inverse, fp64, n, a, 0, lds, nullptr, true);
}

}  // namespace fftb
