// conv_hidden_add_bf16.hip -- instances of the hidden kernel: a residual block's second conv, bf16.
#include "conv_hidden_kernel.h"

namespace pd {

template <>
hipError_t launch_hidden_add<false>(const HiddenCall& c) {
  constexpr bool F8 = false;
  PD_HIDDEN_CASE(64, 64, EPI_ADD)
  PD_HIDDEN_CASE(128, 128, EPI_ADD)
  PD_HIDDEN_CASE(256, 128, EPI_ADD)
  PD_HIDDEN_CASE(512, 128, EPI_ADD)
  return hipErrorInvalidValue;
}

}  // namespace pd
