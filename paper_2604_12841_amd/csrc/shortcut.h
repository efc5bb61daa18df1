// shortcut.h -- the shortcut a residual block adds to its second conv's
// pre-activation, as the conv epilogues read or project it.
#pragma once

#include "activation.h"
#include "internal.h"

namespace pd {

// The projected shortcut of channels co .. co + N - 1 at padded voxel p:
// b[c] + sum_ci w[c][ci] x[p][ci] over the pc channels of x's row (the
// network's input planes, bf16 on both paths), an fp32 FMA chain in channel
// order, rounded to bf16 (F8: to E4M3).
template <int N, bool F8>
__device__ __forceinline__ void project_shortcut(const uint16_t* __restrict__ x, int pc, long long p,
                                                 const float* __restrict__ w, const float* __restrict__ b, int co,
                                                 float (&s)[N]) {
  float a[N];
#pragma unroll
  for (int o = 0; o < N; ++o) a[o] = b[co + o];
  for (int ci = 0; ci < pc; ++ci) {
    const float xv = __uint_as_float((uint32_t)x[p * pc + ci] << 16);
#pragma unroll
    for (int o = 0; o < N; ++o) a[o] = __builtin_fmaf(w[(co + o) * pc + ci], xv, a[o]);
  }
#pragma unroll
  for (int o = 0; o < N; o += 2) {
    if constexpr (F8) {
      s[o] = e4m3_round(a[o]);
      s[o + 1] = e4m3_round(a[o + 1]);
    } else {
      const uint32_t pk = bf16_pack(a[o], a[o + 1]);
      s[o] = __uint_as_float(pk << 16);
      s[o + 1] = __uint_as_float(pk & 0xFFFF0000u);
    }
  }
}

// The block's shortcut of channels co .. co + N - 1 at padded voxel p: its
// stored row in sc (bf16, or F8 E4M3 codes), or with w given its
// projection from sc's few channels (the input planes).
template <int N, bool F8>
__device__ __forceinline__ void shortcut_of(const uint16_t* __restrict__ sc, int sc_stride, long long p,
                                            const float* __restrict__ w, const float* __restrict__ b, int co,
                                            float (&s)[N]) {
  if (w) {
    project_shortcut<N, F8>(sc, sc_stride, p, w, b, co, s);
  } else if constexpr (F8) {
    const uint8_t* r = (const uint8_t*)sc + p * sc_stride + co;
#pragma unroll
    for (int o = 0; o < N; o += 4) {
      const uint32_t q = *reinterpret_cast<const uint32_t*>(r + o);
      s[o] = __builtin_amdgcn_cvt_f32_fp8((int)q, 0);
      s[o + 1] = __builtin_amdgcn_cvt_f32_fp8((int)q, 1);
      s[o + 2] = __builtin_amdgcn_cvt_f32_fp8((int)q, 2);
      s[o + 3] = __builtin_amdgcn_cvt_f32_fp8((int)q, 3);
    }
  } else {
    const uint16_t* r = sc + p * sc_stride + co;
#pragma unroll
    for (int o = 0; o < N; o += 4) {
      const uint2 q = *reinterpret_cast<const uint2*>(r + o);
      s[o] = __uint_as_float(q.x << 16);
      s[o + 1] = __uint_as_float(q.x & 0xFFFF0000u);
      s[o + 2] = __uint_as_float(q.y << 16);
      s[o + 3] = __uint_as_float(q.y & 0xFFFF0000u);
    }
  }
}

}  // namespace pd
