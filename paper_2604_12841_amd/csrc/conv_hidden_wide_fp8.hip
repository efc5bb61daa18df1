// conv_hidden_wide_fp8.hip -- instances of the hidden kernel: activations, 128 output channels, fp8.
#include "conv_hidden_kernel.h"

namespace pd {

template <>
hipError_t launch_hidden_wide<true>(const HiddenCall& c) {
  constexpr bool F8 = true;
  PD_HIDDEN_CASE(128, 128, EPI_ACT)
  PD_HIDDEN_CASE(64, 128, EPI_ACT)
  PD_HIDDEN_CASE(256, 128, EPI_ACT)
  PD_HIDDEN_CASE(512, 128, EPI_ACT)
  return hipErrorInvalidValue;
}

}  // namespace pd
