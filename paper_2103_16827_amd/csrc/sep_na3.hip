// Instantiations of the fused separable module for 1 to 12 four-tap steps.
#include "sep_body.hpp"

namespace qasr {
hipError_t launch_sep_na3(const SepChoice& c, const SepParams& p, size_t lds, hipStream_t st) {
  return sep::launch_na<3>(c, p, lds, st);
}
}  // namespace qasr
