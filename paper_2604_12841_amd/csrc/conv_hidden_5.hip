// conv_hidden_5.hip -- instances of the hidden kernel: 5x5x5 layers (Model 3
// of Table models; bf16, cell tiles only), the output layer included.
#include "conv_hidden_kernel.h"

namespace pd {

hipError_t launch_hidden_5(const HiddenCall& c) {
  const int cout = c.cout == 4 ? 32 : c.cout;  // the output layer's 4 filters fill one padded block
#define PD_HIDDEN_CASE5(CI, CO, E)                                                       \
  if (c.ks == 5 && c.cin == CI && cout == CO && c.epi == E && c.tl->mode == 1)           \
    return launch_one<CI, CO, E, 1, false, 5>(c);
  PD_HIDDEN_CASE5(64, 64, EPI_ACT)
  PD_HIDDEN_CASE5(128, 128, EPI_ACT)
  PD_HIDDEN_CASE5(64, 32, EPI_OUT)
  PD_HIDDEN_CASE5(128, 32, EPI_OUT)
#undef PD_HIDDEN_CASE5
  return hipErrorInvalidValue;
}

}  // namespace pd
