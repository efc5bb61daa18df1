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
  const uint16_t* sc;
  int sc_stride, ks;
  int lsl;          // 2^lsl output-channel slices of c_out channels in one launch
  uint32_t* sched;  // the unit counters, or null
  hipStream_t stream;
  int slice_width = 0;  // small-launch kernel: output channels of a slice of wfrag / bias
};

// Runs call c: a k x k x k layer on the zero-halo activations x (c_in in {64,
// 128, 256, 512}), bf16, or fp8 (E4M3 activations and weight codes, bias
// holding, per slice, c_out biases then c_out per-channel weight scales, one
// byte per value in x and y).
//   epi == 0: a hidden layer (2^lsl slices of c_out = 64 or 128 channels)
//             writing y, whose voxel rows are ystride channels apart;
//   epi == 1: a hidden layer whose epilogue applies the 1x1x1 head and the
//             threshold as launch_conv_single does, instead of writing y;
//   epi == 4: a hidden layer with sc's row (sc_stride values apart) added to
//             the pre-activation (residual blocks), or with head_w the
//             projection of sc's row.
// Weight fragments per slice in 16-channel chunks (conv_fragments in
// api.hip; fp8: conv_fragments_fp8 in 32-channel chunks); n_workgroups =
// conv_hidden_workgroups_per_cu() per CU; sched: 256 zeroed words (per XCD: a
// grab and a done counter, 64 bytes apart): a launch of more than six units
// per workgroup takes its units after the fixed ones from these counters and
// leaves them zero; null: fixed shares.  ks: kernel size 3, or 5 (cells, a
// halo of two; bf16 c_in = c_out = 64 or 128, epi 0).
hipError_t launch_conv_hidden(const HiddenCall& c, bool fp8);

// Whether a launch of nunits units on nwg workgroups takes units from
// counters: from six units per workgroup on.  A unit is taken two ahead, so in
// a short launch the units past the fixed ones all go to the workgroups that
// started first, often both of one CU, while fixed shares spread them over the
// CUs.  With counters from two / six units on: 1100 units of 256-wide layers
// (Model 5 at d = 13, batch 64) 1891 / 1640 us, 1203 units in fp8 (Model 4 at d
// = 13, batch 140) 694 / 631; from three on 2 % more than from six at five and
// a half units (Model 4 at d = 13, batch 330), and no difference past six.
inline bool conv_hidden_counts(long long nunits, long long nwg) { return nunits > 6 * nwg; }

// hipErrorInvalidValue for a call whose instance is not in the unit.
template <bool F8>
hipError_t launch_hidden_narrow(const HiddenCall& c);  // activations, 64 output channels
template <bool F8>
hipError_t launch_hidden_wide(const HiddenCall& c);  // activations, 128 output channels (per slice)
template <bool F8>
hipError_t launch_hidden_head(const HiddenCall& c);  // a fused head
template <bool F8>
hipError_t launch_hidden_add(const HiddenCall& c);  // a shortcut added (residual networks)
hipError_t launch_hidden_5(const HiddenCall& c);  // 5x5x5 layers (bf16)

}  // namespace pd
