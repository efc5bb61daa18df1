// conv_hidden.hip -- the host side of the hidden kernel (conv_hidden_kernel.h):
// its limits, the checks of a call and the dispatch to the unit that holds
// its instance.
#include "conv_hidden_kernel.h"

namespace pd {

int conv_hidden_max_span(int ks) { return ks == 5 ? Conv<5>::MAX_SPAN : Conv<3>::MAX_SPAN; }
int conv_hidden_workgroups_per_cu(int ks) { return ks == 5 ? Conv<5>::WG_PER_CU : Conv<3>::WG_PER_CU; }

hipError_t launch_conv_hidden(const HiddenCall& c, bool fp8) {
  const Geom& g = *c.g;
  const Tiling& tl = *c.tl;
  if (c.ks != 3 && c.ks != 5) return hipErrorInvalidValue;
  if (tl.span <= 0 || tl.span > conv_hidden_max_span(c.ks)) return hipErrorInvalidValue;
  // a shortcut projected in the epilogue: from at most 8 channels of sc
  if (c.epi == EPI_ADD && c.head_w && (!c.head_b || !c.sc || c.sc_stride < 1 || c.sc_stride > 8))
    return hipErrorInvalidValue;
  // the halo holds every tap: a 5x5x5 layer needs the two-voxel halo (and cells)
  if ((c.ks - 1) / 2 > g.pad || (tl.mode == 0 && g.pad != 1)) return hipErrorInvalidValue;
  // output-channel slices: of activation layers (a head needs every channel of a voxel in one unit)
  if (c.lsl < 0 || (1 << c.lsl) > kMaxSlices || (c.lsl > 0 && c.epi == EPI_HEAD)) return hipErrorInvalidValue;
  if (c.ks == 5) return fp8 ? hipErrorInvalidValue : launch_hidden_5(c);
  if (c.epi == EPI_HEAD) return fp8 ? launch_hidden_head<true>(c) : launch_hidden_head<false>(c);
  if (c.epi == EPI_ADD) return fp8 ? launch_hidden_add<true>(c) : launch_hidden_add<false>(c);
  if (c.cout == 128) return fp8 ? launch_hidden_wide<true>(c) : launch_hidden_wide<false>(c);
  return fp8 ? launch_hidden_narrow<true>(c) : launch_hidden_narrow<false>(c);
}

}  // namespace pd
