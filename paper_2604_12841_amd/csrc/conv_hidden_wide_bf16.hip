// conv_hidden_wide_bf16.hip -- instances of the hidden kernel: activations, 128 output channels, bf16.
#include "conv_hidden_kernel.h"

namespace pd {

template <>
hipError_t launch_hidden_wide<false>(const HiddenCall& c) {
  constexpr bool F8 = false;
  PD_HIDDEN_CASE(128, 128, EPI_ACT)
  PD_HIDDEN_CASE(64, 128, EPI_ACT)
  PD_HIDDEN_CASE(256, 128, EPI_ACT)
  PD_HIDDEN_CASE(512, 128, EPI_ACT)
  return hipErrorInvalidValue;
}

}  // namespace pd
