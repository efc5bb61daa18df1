// conv_hidden.h -- what the translation units of the hidden kernel share: a
// call of launch_conv_hidden and the functions that launch it, each holding
// part of the kernel's instances (one unit with all of them compiles for
// minutes).
#pragma once

#include "internal.h"

namespace pd {

struct HiddenCall {
  const Geom* g;
  const Tiling* tl;
  int cin, cout, act;
  const void* x;
  void* y;
  int ystride;
  const void* wfrag;
  const float* bias;
  int epi;  // launch_conv_hidden's `head`
  const float *head_w, *head_b;
  const int32_t* tables;
  uint8_t* nib;
  float* logits;
  int batch, n_workgroups;
  const Split_k* sk;
  const uint16_t* sc;
  int sc_stride, ks;
  hipStream_t stream;
};

// hipErrorInvalidValue for a call whose instance is not in the unit.
template <bool F8>
hipError_t launch_hidden_narrow(const HiddenCall& c);  // activations, 32 or 64 output channels (per slice)
template <bool F8>
hipError_t launch_hidden_wide(const HiddenCall& c);  // activations, 128 output channels (per slice)
template <bool F8>
hipError_t launch_hidden_head(const HiddenCall& c);  // a fused head
template <bool F8>
hipError_t launch_hidden_add(const HiddenCall& c);  // a shortcut added (residual networks)
hipError_t launch_hidden_5(const HiddenCall& c);  // 5x5x5 layers, the output layer included (bf16)

}  // namespace pd
