// conv_hidden_head_fp8.hip -- instances of the hidden kernel: a fused 1x1x1 head, fp8.
#include "conv_hidden_kernel.h"

namespace pd {

template <>
hipError_t launch_hidden_head<true>(const HiddenCall& c) {
  constexpr bool F8 = true;
  PD_HIDDEN_CASE(64, 64, EPI_HEAD)
  PD_HIDDEN_CASE(128, 128, EPI_HEAD)
  PD_HIDDEN_CASE(64, 128, EPI_HEAD)
  PD_HIDDEN_CASE(128, 64, EPI_HEAD)
  return hipErrorInvalidValue;
}

}  // namespace pd
