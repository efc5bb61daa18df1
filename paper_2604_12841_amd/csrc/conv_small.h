// conv_small.h -- the small-launch kernel's interface (conv_small.hip).
#pragma once

#include "conv_hidden.h"

namespace pd {

// Staged lines a tile may need.
constexpr int conv_small_span(int ks) { return ks == 3 ? 512 : 1024; }

// Workgroups per CU: two while the registers and the LDS allow (one: the input
// row is a single piece, 128 bytes; acc: accumulator registers of a lane).
constexpr int conv_small_occupancy(int ks, bool one, int acc) {
  return ks == 3 && acc <= (one ? 64 : 32) ? 2 : 1;
}

// A tile shape, and the K parts of every sum (a power of two that divides the
// layer's 32-byte chunks; fp8: free).
struct SmallPlan {
  int rows, cols, parts;
};

// Everything the kernel needs, as scalars it loads at once at its start (a
// kernel argument that is loaded where it is first used costs that place a
// trip to memory: 0.5 us each on the chain of a small launch).
struct SmallArgs {
  const char* x;
  const void* wfrag;
  char* y;
  const float* bias;
  const float *head_w, *head_b;
  const uint16_t* sc;
  long long S, xbytes;     // padded voxels of a sample; bytes of x
  int T, H, Wp, P;
  // cell tiling (rows and line space as in Tiling, mode 1): cells, tiles, and
  // reciprocals of the sizes divided by (floats: the quotients are small)
  int BI, BJ, sa, sb, span, ntI, ntJ, per, bij;
  float r_sa, r_sb, r_bij, r_bj;
  FastDiv by_ncg, by_per, by_ij, by_j, by_bij, by_bj;
  int ncg;          // channel groups of the layer
  int act;
  int row, np;      // bytes of an input voxel row, staged pieces of it
  int part_chunks;  // chunks of a K part (bf16)
  int ystride;      // channels between output voxel rows
  int nbt, lnbt, tsteps;  // fragments' slices: 32-channel blocks (2^lnbt) and k-steps of one
  int sc_stride;
  // head
  Geom g;
  const int32_t* tables;
  uint8_t* nib;
  float* logits;
};

// Runs call c (c_out: the layer's whole width; epi as in launch_conv_hidden,
// or 2, the 5x5x5 output layer; a head needs cols == c_out) on tiles of pl,
// c.tl a mode 1 tiling of tiles of pl.rows voxels.  c.slice_width: output
// channels of a slice of c.wfrag / c.bias.  Shapes: 1 part 64 x 64, 128 x 64,
// 128 x 128; 2 parts 64 x 32, 64 x 64, 128 x 64, 96 x 128 (rows of more than
// 128 bytes); 4 parts 64 x 32, 64 x 64,
// 128 x 32; more 64 x 32, 64 x 64; fp8 64 x 32, 64 x 64, 128 x 64.
hipError_t launch_conv_small(const SmallPlan& pl, const HiddenCall& c, bool fp8);

}  // namespace pd
