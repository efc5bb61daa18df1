// conv_hidden.hip -- the host side of the hidden kernel (conv_hidden_kernel.h):
// its limits, the checks of a call and the dispatch to the unit that holds
// its instance.
#include "conv_hidden_kernel.h"

namespace pd {

int conv_hidden_max_span(int ks) { return ks == 5 ? Conv<5>::MAX_SPAN : Conv<3>::MAX_SPAN; }
size_t conv_hidden_partial_floats_per_unit() { return (size_t)kTileRows * 128; }
int conv_hidden_workgroups_per_cu(int ks) { return ks == 5 ? Conv<5>::WG_PER_CU : Conv<3>::WG_PER_CU; }

hipError_t launch_conv_hidden(const Geom& g, const Tiling& tl, int cin, int cout, int act, const void* x,
                              void* y, int ystride, const void* wfrag, const float* bias, int head,
                              const float* head_w, const float* head_b, const int32_t* tables, uint8_t* nib,
                              float* logits, int batch, int n_workgroups, const Split_k& sk, int fp8,
                              const uint16_t* sc, int sc_stride, int ks, hipStream_t stream) {
  if (ks != 3 && ks != 5) return hipErrorInvalidValue;
  if (tl.span <= 0 || tl.span > conv_hidden_max_span(ks)) return hipErrorInvalidValue;
  // a shortcut projected in the epilogue: from at most 8 channels of sc
  if (head == 4 && head_w && (!head_b || !sc || sc_stride < 1 || sc_stride > 8)) return hipErrorInvalidValue;
  // the halo holds every tap: a 5x5x5 layer needs the two-voxel halo (and cells)
  if ((ks - 1) / 2 > g.pad || (tl.mode == 0 && g.pad != 1)) return hipErrorInvalidValue;
  // parts per tile: a power of two dividing the layer's chunks, with room
  // for every unit's sums
  const int nchunk = cin / (fp8 ? Prec<true, 3>::KCH : Prec<false, 3>::KCH);
  if (sk.kshift < 0 || nchunk % (1 << sk.kshift) != 0 ||
      (sk.kshift > 0 && (tl.ntiles << (sk.kshift + sk.lsl)) > sk.max_units))
    return hipErrorInvalidValue;
  // output-channel slices: up to max_slices, of activation layers, or of 32
  // or 64 channels for a head (whose rows the second kernel finishes; an
  // output layer needs every channel of a voxel in one unit)
  const bool head_slices = head == EPI_HEAD && (cout == 32 || (cout == 64 && sk.lsl > 0));
  if (sk.lsl < 0 || (1 << sk.lsl) > max_slices(cout) ||
      (sk.lsl > 0 && head != EPI_ACT && head != EPI_ADD && !head_slices))
    return hipErrorInvalidValue;
  // a sliced head parks every unit's sums, also with whole K loops
  if (head_slices && (!sk.partial || (tl.ntiles << (sk.kshift + sk.lsl)) > sk.max_units)) return hipErrorInvalidValue;
  const HiddenCall c{&g,   &tl,    cin,    cout, act,   x,            y,   ystride, wfrag,     bias, head,  head_w,
                     head_b, tables, nib, logits, batch, n_workgroups, &sk, sc,      sc_stride, ks,   stream};
  if (ks == 5) return fp8 ? hipErrorInvalidValue : launch_hidden_5(c);
  if (head == EPI_HEAD) return fp8 ? launch_hidden_head<true>(c) : launch_hidden_head<false>(c);
  if (head == EPI_ADD) return fp8 ? launch_hidden_add<true>(c) : launch_hidden_add<false>(c);
  if (cout == 128) return fp8 ? launch_hidden_wide<true>(c) : launch_hidden_wide<false>(c);
  return fp8 ? launch_hidden_narrow<true>(c) : launch_hidden_narrow<false>(c);
}

int conv_hidden_chunk_channels(int fp8) { return fp8 ? Prec<true, 3>::KCH : Prec<false, 3>::KCH; }

}  // namespace pd
