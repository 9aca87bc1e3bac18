// Instantiations of the fused separable module for 17 to 20 four-tap steps.
#include "sep_body.hpp"

namespace qasr {
hipError_t launch_sep_na5(const SepChoice& c, const SepParams& p, size_t lds, hipStream_t st) {
  return sep::launch_na<5>(c, p, lds, st);
}
}  // namespace qasr
