// Instantiations of the fused separable module for 21 to 24 four-tap steps.
#include "sep_body.hpp"

namespace qasr {
hipError_t launch_sep_na6(const SepChoice& c, const SepParams& p, size_t lds, hipStream_t st) {
  return sep::launch_na<6>(c, p, lds, st);
}
}  // namespace qasr
