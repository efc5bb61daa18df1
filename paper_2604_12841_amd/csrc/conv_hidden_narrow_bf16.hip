// conv_hidden_narrow_bf16.hip -- instances of the hidden kernel: activations, 64 output channels, bf16.
#include "conv_hidden_kernel.h"

namespace pd {

template <>
hipError_t launch_hidden_narrow<false>(const HiddenCall& c) {
  constexpr bool F8 = false;
  PD_HIDDEN_CASE(64, 64, EPI_ACT)
  PD_HIDDEN_CASE(128, 64, EPI_ACT)
  PD_HIDDEN_CASE(256, 64, EPI_ACT)
  return hipErrorInvalidValue;
}

}  // namespace pd
