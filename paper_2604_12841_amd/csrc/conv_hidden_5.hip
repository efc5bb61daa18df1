// conv_hidden_5.hip -- instances of the hidden kernel: 5x5x5 layers (Model 3
// of Table models; bf16, cell tiles only).
#include "conv_hidden_kernel.h"

namespace pd {

hipError_t launch_hidden_5(const HiddenCall& c) {
  if (c.tl->mode != 1 || c.epi != EPI_ACT) return hipErrorInvalidValue;
  if (c.cin == 64 && c.cout == 64) return launch_one<64, 64, EPI_ACT, 1, false, 5>(c);
  if (c.cin == 128 && c.cout == 128) return launch_one<128, 128, EPI_ACT, 1, false, 5>(c);
  return hipErrorInvalidValue;
}

}  // namespace pd
