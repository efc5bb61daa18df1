// conv_hidden_narrow_fp8.hip -- instances of the hidden kernel: activations, 64 output channels, fp8.
#include "conv_hidden_kernel.h"

namespace pd {

template <>
hipError_t launch_hidden_narrow<true>(const HiddenCall& c) {
  constexpr bool F8 = true;
  PD_HIDDEN_CASE(64, 64, EPI_ACT)
  PD_HIDDEN_CASE(128, 64, EPI_ACT)
  PD_HIDDEN_CASE(256, 64, EPI_ACT)
  return hipErrorInvalidValue;
}

}  // namespace pd
