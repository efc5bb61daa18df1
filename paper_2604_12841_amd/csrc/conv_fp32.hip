// conv_fp32.hip -- one 3x3x3 conv3d layer in fp32 end to end (Sec. IV.B, Fig.
// ConvArch; stride 1, zero padding, cross-correlation) as an implicit GEMM on
// the fp32 matrix cores, v_mfma_f32_16x16x4_f32, with bias and activation
// fused in, and for the last hidden layer the 1x1x1 head and the threshold.
// Same zero-halo NTHWC layout as the bf16 path, so every tap is an index
// shift and the K loop has no bounds checks.
//
//   out[co][m] = act(bias[co] + sum_{tap, ci} W[co][ci][tap] * X[m + shift(tap)][ci])
//
// Order of the sums: one fma chain per output, from the bias over the taps
// and, within a tap, the input channels in order; a logit from the head's bias
// over its channels in order.  The instruction is a chain of four fmas in k
// order (bit for bit on 4 M random outputs, subnormal ones among them), so
// results are a scalar loop's, whatever the tiles and the batch, and a logit
// near zero keeps its sign.
//
// Rows are output channels (A, weights), columns output voxels (B).  Lane l
// of an operand holds k = l / 16 of a k-step of 4, so k-step s of a 16-channel
// chunk needs channel 4 s + l / 16 there.  For a lane to read its channels of
// four k-steps with one 16-byte load, a voxel's row is stored with channel 4 s
// + g of a chunk in place 4 g + s (stored_channel); the layer before writes
// that order by taking its own weight rows and biases in it.  (c_in an odd
// multiple of 8: chunks of 8 channels, 8-byte loads, two k-steps, channel 4 s
// + g in place 2 g + s.)  Layer 1 (c_in = 2): k runs over (tap, channel), a
// k-step takes two taps.
//
// Work split: a wave owns MB blocks of 16 consecutive interior voxels x NB
// blocks of 16 output channels and shares nothing with other waves: no LDS,
// no barriers.  Operands come through L1, which holds the 27-fold reuse of a
// wave's footprint; per 16-channel chunk a wave loads (MB + NB) KB for
// MB NB x 4 MFMAs of 32 cycles, so 4 x 4 blocks need 16 bytes per cycle and
// CU of L1's 64, 1 x 1 blocks 64.  Loads run DEPTH - 1 chunks ahead through a
// register ring.  Every load of a layer has one width: with a remainder of 8
// channels loaded on a branch of its own, the compiler waited for the loads
// just issued at the branches' join (249 against 214 us).
//
// Bound: the fp32 matrix rate (157 TFLOP/s) on large launches, load latency
// and L1 on small ones.  Measured: a 64 -> 64 layer of 115200 voxels (d = 9,
// batch 128) 1640 -> 214 us (119 TFLOP/s; 1800 waves of 4 x 4 blocks on 1024
// SIMDs), a 32 -> 32 layer of 11520 voxels (d = 5, batch 64) 109 -> 14 us,
// against one thread per voxel and 8 channels with vector FMAs before.
#include <algorithm>
#include <type_traits>
#include <vector>

#include "internal.h"

namespace pd {
namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

constexpr int MAX_WAVES = 4;  // waves per workgroup at most (independent of each other)
constexpr uint32_t kRange = 0x7FFFFFF0u;  // buffer range in bytes; every offset of a wave is far below

__device__ __forceinline__ float activation_f32(float y, int act) {
  if (act == 1) {  // GELU, tanh form: y / (1 + exp(-2u)), u = sqrt(2/pi)(y + 0.044715 y^3)
    const float k0 = 0.7978845608028654f;
    const float kl = -2.0f * 1.4426950408889634f;
    float u = k0 * (y + 0.044715f * y * y * y);
    float e = __builtin_amdgcn_exp2f(kl * u);
    return y / (1.0f + e);
  }
  if (act == 2) return y > 0.0f ? y : 0.0f;
  return y;
}

// Divisors of the interior-voxel decode u -> (b, t, i, j), and of a wave
// index by the channel groups.
struct Decode {
  FastDiv by_v, by_hh, by_h, by_cg;
};

__device__ __forceinline__ uint32_t uniform(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }

// FIRST: c_in = 2, per-lane taps.  HEAD: the wave holds every channel of its
// voxels (NB blocks cover c_out) and writes the head's logits and nibbles
// instead of y.  bias: of the rows in order (conv_fp32_bias).
// C8: chunks of 8 input channels instead of 16 (c_in an odd multiple of 8).
template <int MB, int NB, int DEPTH, bool FIRST, bool C8, bool HEAD>
__global__ void __launch_bounds__(64 * MAX_WAVES)
    conv_fp32_kernel(Geom g, Decode dc, int cin, int cout, int act, const float* __restrict__ x, float* __restrict__ y,
                     const u32x4* __restrict__ wfrag, uint32_t wbytes, const float* __restrict__ bias,
                     const float* __restrict__ head_w, const float* __restrict__ head_b,
                     const int32_t* __restrict__ tables, uint8_t* __restrict__ nib, float* __restrict__ logits,
                     int nvox, int ncg) {
  const int lane = threadIdx.x & 63, l16 = lane & 15, grp = lane >> 4;
  // (voxel group, channel group) of this wave; a workgroup's waves run over
  // the channel groups first, whose activations L1 then serves once
  const uint32_t wid = blockIdx.x * (blockDim.x >> 6) + uniform(threadIdx.x >> 6);
  const int vg = (int)fdiv(wid, dc.by_cg), cg = (int)wid - vg * ncg;
  const int u0 = vg * 16 * MB;
  if (u0 >= nvox) return;
  const int HH = g.H * g.H;
  auto coords = [&](int u, int& b, int& t, int& i, int& j) {
    b = (int)fastdiv((uint32_t)u, dc.by_v);
    const int v = u - b * g.V;
    t = (int)fdiv((uint32_t)v, dc.by_hh);
    const int s = v - t * HH;
    i = (int)fastdiv((uint32_t)s, dc.by_h);
    j = s - i * g.H;
  };
  // padded voxel of each block's lane (past the end: the last voxel, not
  // stored), and the wave's base: the (0, 0, 0) tap of its first voxel
  int pv[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    int b, t, i, j;
    coords(min(u0 + 16 * mb + l16, nvox - 1), b, t, i, j);
    pv[mb] = (int)padded_index(g, b, t, i, j);
  }
  const int p0 = (int)uniform((uint32_t)pv[0]);
  const int corner = g.P + g.Wp + 1;  // from a voxel back to its (0, 0, 0) tap
  const float* const xb = x + (long long)(p0 - corner) * cin;
  const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc((void*)xb, 0, kRange, 0x00020000);
  const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc((void*)wfrag, 0, wbytes, 0x00020000);
  uint32_t voff[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) voff[mb] = (uint32_t)((pv[mb] - p0) * cin) * 4u;

  const int nbt = (cout + 15) >> 4;  // channel blocks of the layer
  f32x4 acc[MB][NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {  // lane: rows 4 grp .. + 3 of the block (past the last block: no rows)
    const int row = (cg * NB + nb) * 16 + grp * 4;
    const f32x4 b0 = row < nbt * 16 ? *reinterpret_cast<const f32x4*>(bias + row) : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) acc[mb][nb] = b0;
  }

  if constexpr (FIRST) {
    // fragment m: lane l's weights of two k-steps, 2 m and 2 m + 1; a k-step s is taps 2 s and 2 s + 1 (lane l: tap
    // 2 s + l / 32, channel (l / 16) % 2)
#pragma unroll
    for (int m = 0; m < 7; ++m) {
      u32x2 av[NB];
      uint32_t bv[MB][2];
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int t0 = 4 * m + 2 * s, t1 = t0 < 26 ? t0 + 1 : t0;  // the tap past the last: weights of -0, which add nothing
        const int o0 = (t0 / 9) * g.P + (t0 / 3) % 3 * g.Wp + t0 % 3, o1 = (t1 / 9) * g.P + (t1 / 3) % 3 * g.Wp + t1 % 3;
        const uint32_t to = (uint32_t)((grp >> 1 ? o1 : o0) * 2 + (grp & 1)) * 4u;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) bv[mb][s] = __builtin_amdgcn_raw_buffer_load_b32(xr, voff[mb] + to, 0, 0);
      }
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        av[nb] = __builtin_amdgcn_raw_buffer_load_b64(wr, lane * 8u, (uint32_t)((m * nbt + cg * NB + nb) * 512), 0);
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb)
            acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(av[nb][s]), __uint_as_float(bv[mb][s]),
                                                               acc[mb][nb], 0, 0, 0);
    }
  } else {
    constexpr int KC = C8 ? 8 : 16;    // input channels of a chunk
    constexpr int KS = KC / 4;         // its k-steps, channels per lane
    const int nch = cin / KC;          // chunks of a tap
    const int niter = 27 * nch;        // a multiple of DEPTH
    typedef __attribute__((ext_vector_type(KS))) uint32_t frag;
    frag bq[DEPTH][MB], aq[DEPTH][NB];
    // the iteration loaded next, its chunk and tap (scalars; past the last
    // iteration the last one is loaded again)
    int li = 0, lc = 0, lt = 0;
    auto load = [&](frag (&bv)[MB], frag (&av)[NB]) {
      const int dt = lt / 9, di = (lt / 3) % 3, dj = lt % 3;
      const uint32_t so = (uint32_t)((dt * g.P + di * g.Wp + dj) * cin + lc * KC) * 4u;
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        if constexpr (C8) bv[mb] = __builtin_amdgcn_raw_buffer_load_b64(xr, voff[mb] + grp * 8u, so, 0);
        else bv[mb] = __builtin_amdgcn_raw_buffer_load_b128(xr, voff[mb] + grp * 16u, so, 0);
      }
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const uint32_t wo = (uint32_t)((li * nbt + cg * NB + nb) * (64 * KC));
        if constexpr (C8) av[nb] = __builtin_amdgcn_raw_buffer_load_b64(wr, lane * 8u, wo, 0);
        else av[nb] = __builtin_amdgcn_raw_buffer_load_b128(wr, lane * 16u, wo, 0);
      }
      if (li + 1 < niter) {
        ++li;
        if (++lc == nch) {
          lc = 0;
          ++lt;
        }
      }
    };
#pragma unroll
    for (int d = 0; d < DEPTH - 1; ++d) load(bq[d], aq[d]);
    for (int it = 0; it < niter; it += DEPTH) {
#pragma unroll
      for (int d = 0; d < DEPTH; ++d) {
        load(bq[(d + DEPTH - 1) % DEPTH], aq[(d + DEPTH - 1) % DEPTH]);
        __builtin_amdgcn_sched_barrier(0);  // the loads go out before this iteration's MFMAs
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
          for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
              acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(aq[d][nb][s]),
                                                                 __uint_as_float(bq[d][mb][s]), acc[mb][nb], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }

  // Lane holds rows 16 (cg NB + nb) + 4 grp .. + 3, in that place of voxel u0 + 16 mb + l16.
  if constexpr (HEAD) {
    // Value e of a lane is channel 16 nb + 4 e + grp (conv_fp32_fragments): the
    // B operand of the head's k-step of channels 16 nb + 4 e .. + 3.  Rows 0..3
    // of A are the head's filters.
    f32x4 lg[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int o = 0; o < 4; ++o) lg[mb][o] = grp == 0 ? head_b[o] : 0.0f;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int c = nb * 16 + e * 4;
        if (c < cout) {  // uniform
          const float hw = l16 < 4 ? head_w[l16 * cout + c + grp] : 0.0f;
#pragma unroll
          for (int mb = 0; mb < MB; ++mb)
            lg[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(hw, activation_f32(acc[mb][nb][e], act), lg[mb], 0, 0, 0);
        }
      }
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const int u = u0 + 16 * mb + l16;
      if (u < nvox && grp == 0) {
        int b, t, i, j;
        coords(u, b, t, i, j);
        const float l4[4] = {lg[mb][0], lg[mb][1], lg[mb][2], lg[mb][3]};
        nib[u] = (uint8_t)flip_nibble(g, tables, i, j, l4);
        if (logits) {
#pragma unroll
          for (int o = 0; o < 4; ++o) logits[(((long long)b * 4 + o) * g.T + t) * HH + i * g.H + j] = l4[o];
        }
      }
    }
  } else {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int co = (cg * NB + nb) * 16 + grp * 4;
      if (co < cout) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
          f32x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = activation_f32(acc[mb][nb][e], act);
          if (u0 + 16 * mb + l16 < nvox) *reinterpret_cast<f32x4*>(y + (long long)pv[mb] * cout + co) = v;
        }
      }
    }
  }
}

// k-steps of a chunk of a c-channel row (c a multiple of 8).
inline int chunk_steps(int c) { return c % 16 ? 2 : 4; }

// Channel in place p of a row stored in chunks of n k-steps: channel 4 s + g of a chunk lies in place n g + s.
inline int stored_channel(int p, int n) {
  const int q = p % (4 * n);
  return p - q + 4 * (q % n) + q / n;
}

// Output channel of weight row r: the place it is stored in, by the chunks
// of the next layer; a head's layer stores nothing and takes chunks of 16.
inline int row_channel(int r, int cout, int head) { return stored_channel(r, head ? 4 : chunk_steps(cout)); }

}  // namespace

// Fragments of an fp32 layer: [iteration][block of 16 rows][64 lanes][n]
// floats, iterations (tap, chunk of 4 n input channels), n = chunk_steps:
// lane l holds channels 4 n chunk + 4 s + l / 16, s = 0 .. n - 1, of row 16
// block + l % 16.  c_in = 2: 7 iterations, n = 2, over k = 2 tap + channel:
// lane l holds k = 8 iteration + 4 s + l / 16 (past the last tap -0: the
// events are 0 or 1, and a sum plus -0 is the sum).  Rows that do not exist
// are zero.
std::vector<float> conv_fp32_fragments(const float* w, int cin, int cout, int head) {
  const int nbt = (cout + 15) / 16, n = cin == 2 ? 2 : chunk_steps(cin);
  const int nch = cin / (4 * n), niter = cin == 2 ? 7 : 27 * nch;
  std::vector<float> f((size_t)niter * nbt * 64 * n, 0.0f);
  for (int it = 0; it < niter; ++it)
    for (int nb = 0; nb < nbt; ++nb)
      for (int l = 0; l < 64; ++l) {
        const int co = row_channel(nb * 16 + l % 16, cout, head);
        if (co >= cout) continue;
        for (int s = 0; s < n; ++s) {
          const int k = 8 * it + 4 * s + l / 16;
          const int tap = cin == 2 ? k / 2 : it / nch, ci = cin == 2 ? k % 2 : (it % nch) * 4 * n + 4 * s + l / 16;
          f[(((size_t)it * nbt + nb) * 64 + l) * n + s] = tap < 27 ? w[((size_t)co * cin + ci) * 27 + tap] : -0.0f;
        }
      }
  return f;
}

// Biases of the rows of an fp32 layer, in whole blocks of 16.
std::vector<float> conv_fp32_bias(const float* b, int cout, int head) {
  std::vector<float> r((size_t)(cout + 15) / 16 * 16, 0.0f);
  for (size_t k = 0; k < r.size(); ++k) {
    const int co = row_channel((int)k, cout, head);
    if (co < cout) r[k] = b[co];
  }
  return r;
}

// Cycles of a 16-channel chunk: m n x 128 of MFMAs, or the four SIMDs' loads
// through the CU's L1, where a block of voxels (16 rows in as many lines)
// takes 64 and a weight block 16 -- 355 cycles were measured for 1 x 1
// blocks.  Times the waves a SIMD runs one after the other; of equals the
// larger tile.  A head needs all channel blocks in the wave (4 x 4 or 2 x 8
// blocks fit the registers).
Fp32Blocks conv_fp32_blocks(long long nvox, int cout, int head, int n_cu) {
  const int nbt = (cout + 15) / 16;
  const long long simds = 4ll * n_cu;
  Fp32Blocks r{1, 1, -1};
  for (int m = 1; m <= 4; m *= 2)
    for (int n = 1; n <= 8; ++n) {
      if (m * n > 16 || (head ? n != nbt : n > std::min(nbt, 4))) continue;
      const long long waves = (nvox + 16 * m - 1) / (16 * m) * ((nbt + n - 1) / n);
      const long long cost = (waves + simds - 1) / simds * std::max(128 * m * n, 4 * (64 * m + 16 * n));
      if (r.cost < 0 || cost < r.cost || (cost == r.cost && m * n > r.mb * r.nb)) r = {m, n, cost};
    }
  return r;
}

hipError_t launch_conv_fp32(const Geom& g, int cin, int cout, int act, const float* x, float* y, const float* w,
                            const float* bias, int head, const float* head_w, const float* head_b,
                            const int32_t* tables, uint8_t* nib, float* logits, int batch, int n_cu,
                            hipStream_t stream) {
  if (cout < 8 || cout % 8 != 0 || cout > 128 || (cin != 2 && (cin < 8 || cin % 8 != 0 || cin > 128)) || g.pad != 1)
    return hipErrorInvalidValue;
  const long long nvox = (long long)batch * g.V;  // < 2^31 (host check)
  const int nbt = (cout + 15) / 16;
  const uint32_t wbytes = (uint32_t)(cin == 2 ? 7 * 512 : 27 * 64 * cin) * nbt;
  const long long simds = 4ll * n_cu;
  const Fp32Blocks bl = conv_fp32_blocks(nvox, cout, head, n_cu);
  const int mb = bl.mb, nb = bl.nb;
  hipError_t err = hipErrorInvalidValue;
  auto launch = [&](auto M, auto N, auto F, auto E, auto HD) {
    constexpr int MB = decltype(M)::value, NB = decltype(N)::value;
    if constexpr (MB * NB <= 16 && (NB <= 4 || decltype(HD)::value)) {
      constexpr int DEPTH = MB + NB <= 4 ? 9 : 3;  // ring depth in chunks (divides 27)
      const int ncg = (nbt + NB - 1) / NB;
      Decode dc;
      dc.by_v = make_fastdiv((uint32_t)g.V);
      dc.by_hh = make_fastdiv((uint32_t)(g.H * g.H));
      dc.by_h = make_fastdiv((uint32_t)g.H);
      dc.by_cg = make_fastdiv((uint32_t)ncg);
      const long long waves = (nvox + 16 * MB - 1) / (16 * MB) * ncg;
      // up to one wave per SIMD: workgroups of one wave, which spread evenly
      // over the CUs and their L1s
      const int wpg = waves <= simds ? 1 : MAX_WAVES;
      if (waves >= (1ll << 31)) return;  // (the error stays: wave numbers are 32-bit)
      hipLaunchKernelGGL((conv_fp32_kernel<MB, NB, DEPTH, decltype(F)::value, decltype(E)::value, decltype(HD)::value>),
                         dim3((unsigned)((waves + wpg - 1) / wpg)), dim3(64 * wpg), 0, stream, g, dc, cin, cout,
                         act, x, y, (const u32x4*)w, wbytes, bias, head_w, head_b, tables, nib, logits, (int)nvox,
                         ncg);
      err = hipGetLastError();
    }
  };
  auto by_size = [&](auto F, auto E, auto HD) {
    auto cols = [&](auto M) {
      switch (nb) {
#define PD_NB(N) \
  case N: launch(M, std::integral_constant<int, N>(), F, E, HD); break;
        PD_NB(1) PD_NB(2) PD_NB(3) PD_NB(4) PD_NB(5) PD_NB(6) PD_NB(7) PD_NB(8)
#undef PD_NB
      }
    };
    if (mb == 1) cols(std::integral_constant<int, 1>());
    if (mb == 2) cols(std::integral_constant<int, 2>());
    if (mb == 4) cols(std::integral_constant<int, 4>());
  };
  auto by_head = [&](auto F, auto E) {
    if (head) by_size(F, E, std::true_type());
    else by_size(F, E, std::false_type());
  };
  if (cin == 2) by_head(std::true_type(), std::false_type());
  else if (cin % 16) by_head(std::false_type(), std::true_type());
  else by_head(std::false_type(), std::false_type());
  return err;
}

}  // namespace pd
