// conv_small.hip -- a 3x3x3 (5x5x5) conv3d layer (Sec. IV.B, Fig. ConvArch) of
// a small launch: the layer of conv_hidden_kernel.h (same weights, precision
// points and epilogues) when its 256-voxel tiles would leave the chip mostly
// idle.  There a layer's time is one workgroup's chain of latencies, not
// matrix work, so this kernel shortens that chain:
//   * A workgroup (4 waves) computes a tile of 64, 96 or 128 voxels x 32
//     to 128 output channels.  Its waves are KG K groups x WM voxel groups x WN
//     channel groups; a wave owns MB x NB blocks of 32 voxels x 32 channels
//     and the consecutive input-channel chunks (32 bytes per voxel) of its K
//     group.  The partial sums meet in LDS, where every lane finishes 8
//     channels of a voxel: sum in part order, bias, activation, one 16-byte
//     store.
//   * The footprint is staged in pieces of four chunks (128 bytes per voxel),
//     no barrier inside a piece, the next piece's loads in flight meanwhile.
//   * Weight fragments run a whole ring ahead, starting before anything else.
//   * Staging addresses come from a table in LDS with one entry per staged
//     line, not from a decode per load.
// The K parts of a sum: an output is the sum, in order, of P parts of
// consecutive chunks, each part one chain of MFMAs (conv_parts in api.hip
// chooses P from the launch's size; KG = min(P, 4); MULTI: P / 4 rounds of four
// parts, each folded into a lane's totals).  fp8 layers always run KG = 4.
// Tiles are cells' runs (mode 1 of Tiling, of R rows), voxels 144 bytes apart
// in LDS (granule g of voxel v in bank group (9 v + g) mod 16: 16 consecutive
// voxels meet no group twice).  Lines outside the grid stage whatever the
// buffer holds there (zeros past its end): they only feed rows that are
// discarded.
// Bound: at one workgroup per CU the chain of latencies -- 1.1 us to the
// first staging loads (kernel arguments, the line table), 1.0 staging, 0.3
// exchanging sums, 0.7 epilogue -- and a K loop at 50-80 % of the matrix rate.
// Measured per layer in us at batch 1, before (256-voxel tiles as output
// slices of 32 or 64 channels, or with K loops split over workgroups and
// finished by a second kernel) and now: 64 channels bf16 d = 13 / 25 / 31 13.5
// / 15.9 / 16.5 -> 5.6 / 11.7 / 11.6, 128 channels bf16 18.5 / 30.0 / 33.0 ->
// 7.4 / 23.8 / 27.1, 128 channels fp8 15.4 / 21.9 / 22.1 -> 5.8 / 16.2 / 19.1;
// a 5x5x5 layer at d = 13 / 21 42.9 / 66.6 -> 24.6 / 62.5.
// Two parts take 96 x 128 tiles (six MFMAs for 2 KB of weights and 3 of
// fragments; 128 x 64 ones four for 2 and 2) where 128 x 64 ones are a few more
// than the CUs: Model 3 at d = 13, batch 8 (its 128-wide 5x5x5 layers, 184
// tiles instead of 288) 250 -> 207 us, Model 6 at 13^3, batch 16 (the last two
// samples of the 512-wide layers) 2740 -> 2545.
// Four parts of 256 channels and more take 96 x 64 tiles where those leave CUs free
// (512 channels: fit them once; 64 x 32 ones are three times as many, two to a CU):
// a wave's nine steps of weights in flight last 0.8 us of MFMAs there, about a first
// read from memory, 64 x 32 tiles' 0.3.  In us, 64 x 32 / 96 x 64 (and 256-voxel tiles with their
// K loops split over workgroups, before this kernel): Model 6 at 13^3, batch 1 417
// / 288 (406), Model 5 at 17^3 163 / 124 (208), Model 2 at 13^3, batch 2 98 / 74 (107).
#include <algorithm>

#include "activation.h"
#include "conv_small.h"
#include "lds_limit.h"
#include "shortcut.h"
#include "tiles.h"

namespace pd {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(8))) uint32_t u32x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(8))) int i32x8;
typedef __attribute__((address_space(3))) char lds_char;
typedef __attribute__((address_space(3))) const u32x4 lds_u32x4;
typedef __attribute__((address_space(3))) u32x4 lds_u32x4_w;
typedef __attribute__((address_space(3))) uint32_t lds_u32_w;
typedef __attribute__((address_space(3))) f32x4 lds_f32x4;

constexpr int NT = 256;           // threads: 4 waves, one chunk of a piece each
constexpr uint32_t kNoLine = 0x80000000u;  // staging offset past every buffer range: loads zeros

// The shape of a workgroup.  HALF: fp8 rows of 64 bytes (64 input channels):
// two chunks, whose steps are halved over two K groups each.  ONE: the row is
// one piece (nothing to prefetch during the K loop).
template <int KS_, bool F8_, bool HALF_, bool ONE_, int KG_, bool MULTI_, int WM_, int WN_, int MB_, int NB_>
struct Small {
  static constexpr int KS = KS_, KG = KG_, WM = WM_, WN = WN_, MB = MB_, NB = NB_;
  static constexpr bool F8 = F8_, HALF = HALF_, ONE = ONE_, MULTI = MULTI_;
  static_assert(KG * WM * WN == 4 && (KG == 4 || !F8) && (KG == 4 || !MULTI), "four waves");
  static constexpr int R = 32 * MB * WM, TC = 32 * NB * WN;
  static constexpr int TAPS = KS * KS * KS;
  static constexpr int SPAN = conv_small_span(KS);
  static constexpr int PB = HALF ? 64 : 128;      // staged bytes per voxel and piece
  static constexpr int VSTR = PB + 16;            // their LDS stride
  static constexpr int CG = 4 / KG;               // chunks of a piece in a K group
  static constexpr int CSTEP = F8 ? (TAPS + 1) / 2 : TAPS;  // k-steps of a chunk
  static constexpr int NSTEP = HALF ? CSTEP / 2 : CSTEP;    // ... that a wave runs
  static constexpr int ACC = 16 * MB * NB;        // accumulator registers
  static constexpr int OCC = conv_small_occupancy(KS, ONE, ACC);
  // weight ring depth (a divisor of NSTEP)
  static constexpr int RING = KS == 5 ? (NB == 1 && MB < 4 ? 25 : 5)
                              : F8    ? (HALF || MB * NB > 2 || !ONE ? 7 : 14)
                                      : (NB == 2 || MB > 2 || (!ONE && MB > 1) ? 9 : 27);
  // steps between a fragment's read and its use: an LDS read takes about 130
  // cycles here, a step's MFMAs 32 MB NB (fp8: 64 MB NB); a divisor of NSTEP
  // where fragments are read on into the next chunk
  static constexpr int AD = KS == 5 ? (CG > 1 ? 5 : (MB * NB <= 2 ? 4 : 2))
                            : F8    ? (MB * NB == 2 ? 3 : 2)
                                    : (MB * NB == 1 && ONE ? 9 : 3);
  static_assert(CG == 1 || NSTEP % AD == 0, "fragments run on into the next chunk");
  static constexpr int WFRAG = F8 ? 2048 : 1024;  // bytes of a weight fragment
  static constexpr int ROUNDS = SPAN * PB / (16 * NT);
  // the K groups' partial sums, over the staging area: [KG][R][TC] fp32, rows padded
  static constexpr int RSTR = TC * 4 + 16;
  static constexpr int table = SPAN * VSTR > KG * R * RSTR ? SPAN * VSTR : KG * R * RSTR;  // [SPAN] staging offsets
  static constexpr int consts = table + SPAN * 4;  // biases [TC], scales [TC], head weights [4][TC]
  static constexpr int lds = consts + 6 * TC * 4;
  static_assert(NSTEP % RING == 0, "the weight ring lines up with chunks");
  static_assert(OCC * lds <= 160 * 1024, "the workgroups of a CU fit its LDS");
};

// u / d for a small u >= 0, r = 1 / d: exact for u < 2^16 and d < 2^10 (the
// quotient of u + 1/2 lies at least 1 / 2d from an integer).
__device__ __forceinline__ int small_div(int u, float r) { return (int)(((float)u + 0.5f) * r); }

// a b + c for factors below 2^24 (a full-rate multiply-add).
__device__ __forceinline__ int mad24(int a, int b, int c) { return (int)__umul24((unsigned)a, (unsigned)b) + c; }

template <typename S, int EPI>
__global__ void __launch_bounds__(NT)
__attribute__((amdgpu_waves_per_eu(S::OCC, S::OCC)))
conv_small_kernel(SmallArgs p) {
  constexpr int KS = S::KS, KG = S::KG, MB = S::MB, NB = S::NB, CG = S::CG, AD = S::AD;
  constexpr bool F8 = S::F8, HALF = S::HALF, ONE = S::ONE, MULTI = S::MULTI;
  constexpr int R = S::R, TC = S::TC, NSTEP = S::NSTEP, RING = S::RING, VSTR = S::VSTR;
  constexpr int HW = (KS - 1) / 2;  // the halo
  constexpr int ESZ = F8 ? 1 : 2;
  constexpr int WQ = F8 ? 2 : 1;  // 16-byte pieces of a fragment's lane
  extern __shared__ __attribute__((aligned(16))) char smem[];
  // all arguments in one go
  asm volatile("" ::"s"(p.x), "s"(p.wfrag), "s"(p.y), "s"(p.bias), "s"(p.S), "s"(p.xbytes), "s"(p.T), "s"(p.H),
               "s"(p.Wp), "s"(p.P), "s"(p.BI), "s"(p.BJ), "s"(p.sa), "s"(p.sb), "s"(p.span), "s"(p.ntJ), "s"(p.per),
               "s"(p.bij), "s"(p.r_sa), "s"(p.r_bij));
  lds_char* const lds = (lds_char*)smem;
  const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, l32 = lane & 31;
  const int wave = (int)__builtin_amdgcn_readfirstlane((uint32_t)tid >> 6);
  const int kg = wave / (S::WM * S::WN), wo = wave % (S::WM * S::WN), wm = wo % S::WM, wn = wo / S::WM;
  // channel groups vary fastest over the workgroups: the 8 XCDs take
  // workgroups in turn, so an XCD's L2 holds the weights of few groups
  const int tile = (int)fdiv(blockIdx.x, p.by_ncg), cg = (int)blockIdx.x - tile * p.ncg;

  // ---- weights: the first ring of this wave's k-steps ----
  // k-step s of chunk c: fragment c CSTEP + s of the layer (HALF: a K group
  // runs half the steps of chunk kg / 2), blocks cb .. cb + NB - 1
  const int nc = ONE ? CG : CG * p.np;          // this wave's chunks
  const int pc = MULTI ? p.part_chunks : nc;    // ... of a round's part: (4 round + kg) pc ..
  const int cb = (cg * S::WN + wn) * NB, slice = cb >> p.lnbt;
  const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc((void*)p.wfrag, 0, 0x7FFFFFF0u, 0x00020000);
  const uint32_t wstep = (uint32_t)p.nbt * S::WFRAG;
  const int gs0 = HALF ? (kg >> 1) * S::CSTEP + (kg & 1) * NSTEP : kg * pc * S::CSTEP;
  uint32_t wbase = (uint32_t)(slice * p.tsteps + gs0) * wstep + (uint32_t)(cb - (slice << p.lnbt)) * S::WFRAG;
  u32x4 bq[RING][NB][WQ];
  auto wload = [&](uint32_t so, u32x4 (&dst)[NB][WQ]) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int h = 0; h < WQ; ++h)
        dst[nb][h] = __builtin_amdgcn_raw_buffer_load_b128(wres, (uint32_t)lane * (16 * WQ) + 16 * h,
                                                           so + (uint32_t)nb * S::WFRAG, 0);
  };
#pragma unroll
  for (int s = 0; s < RING - 1; ++s) wload(wbase + s * wstep, bq[s]);
  __builtin_amdgcn_sched_barrier(0);
  // biases (fp8: and scales; per slice its biases, then its scales), head weights
  typedef __attribute__((address_space(3))) float lds_float;
  lds_float* const consts = (lds_float*)(lds + S::consts);
  const int cw = p.nbt * 32, sl0 = (cg * TC) >> (p.lnbt + 5);  // the tile's slice of the bias array
  const float* const bsl = p.bias + (F8 ? 2 : 1) * sl0 * cw + (cg * TC - sl0 * cw);
  float cv = 0.0f, hv = 0.0f;
  if (tid < (F8 ? 2 : 1) * TC) cv = bsl[tid < TC ? tid : cw + tid - TC];
  if (EPI == 1 && tid < 4 * TC) hv = p.head_w[tid];

  // ---- staging table: byte offset of every staged line from the tile's first ----
  const int b = (int)fdiv((uint32_t)tile, p.by_per), rem = tile - b * p.per;
  const int run = (int)fdiv((uint32_t)rem, p.by_ij), rem2 = rem - run * (p.ntI * p.ntJ);
  const int ti = (int)fdiv((uint32_t)rem2, p.by_j);
  const int i0 = ti * p.BI, j0 = (rem2 - ti * p.ntJ) * p.BJ;
  const int a0 = (int)fdiv((uint32_t)(run * R), p.by_bij), w0 = run * R - a0 * p.bij;
  const int c0 = (int)fdiv((uint32_t)w0, p.by_bj), e0 = w0 - c0 * p.BJ;
  const int line0 = c0 * p.sb + e0, first = c0 * p.Wp + e0;  // within round a0 of the cell
  lds_u32_w* const table = (lds_u32_w*)(lds + S::table);
#pragma unroll
  for (int k = 0; k < S::SPAN / NT; ++k) {
    const int v = k * NT + tid, u = line0 + v;
    const int a = small_div(u, p.r_sa), ur = u - mad24(a, p.sa, 0);
    const int c = small_div(ur, p.r_sb), e = ur - mad24(c, p.sb, 0);
    table[v] = v < p.span ? __umul24((unsigned)(mad24(a, p.P, mad24(c, p.Wp, e)) - first), (unsigned)p.row) : kNoLine;
  }
  if (tid < (F8 ? 2 : 1) * TC) consts[tid] = cv;
  if (EPI == 1 && tid < 4 * TC) consts[2 * TC + tid] = hv;
  const long long origin = (long long)b * p.S + (long long)a0 * p.P + first + (long long)i0 * p.Wp + j0;
  const long long left = p.xbytes - origin * p.row;  // bytes from the origin on
  const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(p.x + origin * p.row), 0, (uint32_t)(left < 0x7FFFFFF0ll ? left : 0x7FFFFFF0ll), 0x00020000);
  // tile row r: its round (from a0), row and column in the cell; whether it is inside the volume
  auto row_of = [&](int r, int& a, int& c, int& e) -> bool {
    const int u = w0 + r;
    a = small_div(u, p.r_bij);
    const int ur = u - mad24(a, p.bij, 0);
    c = small_div(ur, p.r_bj);
    e = ur - mad24(c, p.BJ, 0);
    return a0 + a < p.T && i0 + c < p.H && j0 + e < p.H;
  };
  // rows of this lane: LDS address of the (0,0,0) tap, this wave's chunk
  uint32_t rbase[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    int a, c, e;
    const bool ok = row_of((wm * MB + mb) * 32 + l32, a, c, e);
    const int lb = ok ? mad24(a, p.sa, mad24(c, p.sb, e)) - line0 : 0;
    rbase[mb] = (uint32_t)(uintptr_t)lds + (uint32_t)(lb * VSTR + (HALF ? kg >> 1 : kg * CG) * 32 + (F8 ? 0 : half * 16));
  }
  __syncthreads();

  // a piece: the next CG chunks of every K group, 32 bytes each
  constexpr int G = S::PB / 16;  // granules per voxel and piece
  const int gr = tid % G, slot = gr >> 1;
  const uint32_t goff = (uint32_t)(HALF ? gr * 16 : ((slot / CG) * pc + slot % CG) * 32 + (gr & 1) * 16);
  u32x4 stg[S::ROUNDS];
  auto stage_load = [&](int ch) {  // the piece that starts with the groups' ch-th chunk
    const uint32_t so = (uint32_t)(MULTI ? ch + ch / pc * 3 * pc : ch) * 32;
#pragma unroll
    for (int k = 0; k < S::ROUNDS; ++k) {
      if (k * (NT / G) >= p.span) break;  // uniform
      stg[k] = __builtin_amdgcn_raw_buffer_load_b128(xres, table[(k * NT + tid) / G] + goff, so, 0);
    }
  };
  auto stage_store = [&]() {
#pragma unroll
    for (int k = 0; k < S::ROUNDS; ++k) {
      if (k * (NT / G) >= p.span) break;
      *(lds_u32x4_w*)(lds + (k * NT + tid) / G * VSTR + gr * 16) = stg[k];
    }
  };
  stage_load(0);

  f32x16 acc[MB][NB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[mb][nb][v] = 0.0f;

  const uint32_t hmask = half ? 0xFFFFFFFFu : 0u;
  constexpr int AQ = F8 ? 2 : 1;
  const int tap0 = HALF ? 2 * NSTEP * (kg & 1) : 0;  // first tap of this wave's steps
  int sa = p.sa * VSTR, sb = p.sb * VSTR;
  auto tap_off = [&](int tap) -> uint32_t {
    const int dt = tap / (KS * KS), di = (tap / KS) % KS, dj = tap % KS;
    return (uint32_t)(dt * sa + di * sb + dj * VSTR);
  };
  auto frag_read = [&](int mb, int s, int chunk_off, u32x4 (&dst)[AQ]) {
    // each step computes its own address (none held across the loop)
    asm volatile("" : "+v"(rbase[mb]), "+s"(sa), "+s"(sb));
    if constexpr (F8) {
      uint32_t hm = hmask;
      asm volatile("" : "+v"(hm));
      const int t0 = tap0 + 2 * s, t1 = t0 + 1 < S::TAPS ? t0 + 1 : t0;  // the tap past the last: zero weights
      const uint32_t o0 = tap_off(t0), o1 = tap_off(t1);
      const uint32_t a = rbase[mb] + o0 + ((o1 - o0) & hm) + chunk_off;
      dst[0] = *(lds_u32x4*)(uintptr_t)a;
      dst[AQ - 1] = *(lds_u32x4*)(uintptr_t)(a + 16);
    } else {
      dst[0] = *(lds_u32x4*)(uintptr_t)(rbase[mb] + tap_off(s) + chunk_off);
    }
  };
  auto mfma = [&](const u32x4 (&w)[WQ], const u32x4 (&a)[AQ], f32x16 c) -> f32x16 {
    if constexpr (F8) {
      const i32x8 wa = __builtin_bit_cast(
          i32x8, u32x8{w[0].x, w[0].y, w[0].z, w[0].w, w[WQ - 1].x, w[WQ - 1].y, w[WQ - 1].z, w[WQ - 1].w});
      const i32x8 ab = __builtin_bit_cast(
          i32x8, u32x8{a[0].x, a[0].y, a[0].z, a[0].w, a[AQ - 1].x, a[AQ - 1].y, a[AQ - 1].z, a[AQ - 1].w});
      return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(wa, ab, c, 0, 0, 0, 0, 0, 0);
    } else {
      return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w[0]), __builtin_bit_cast(bf16x8, a[0]),
                                                     c, 0, 0, 0);
    }
  };

  // this wave's partial sums into LDS, and a pass's row of all of them, added
  // in order to v (of the first round: set)
  auto put_sums = [&]() {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *(lds_f32x4*)(lds + (kg * R + (wm * MB + mb) * 32 + l32) * S::RSTR +
                        ((wn * NB + nb) * 32 + q * 8 + half * 4) * 4) =
              f32x4{acc[mb][nb][4 * q], acc[mb][nb][4 * q + 1], acc[mb][nb][4 * q + 2], acc[mb][nb][4 * q + 3]};
  };
  constexpr int GPR = TC / 8, RPW = 64 / GPR;  // lanes per row, rows per wave and pass
  constexpr int PASSES = R / (4 * RPW);
  const int grp = lane % GPR;
  auto get_sums = [&](int ps, bool first_round, float (&v)[8]) {
    const int r = (ps * 4 + wave) * RPW + lane / GPR;
#pragma unroll
    for (int w = 0; w < KG; ++w) {
      const lds_char* src = lds + (w * R + r) * S::RSTR + grp * 32;
      const f32x4 lo = *(const lds_f32x4*)src, hi = *(const lds_f32x4*)(src + 16);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[e] = w == 0 && first_round ? lo[e] : v[e] + lo[e];
        v[4 + e] = w == 0 && first_round ? hi[e] : v[4 + e] + hi[e];
      }
    }
  };
  float tot[MULTI ? PASSES : 1][8];

  // ---- K loop: this wave's chunks, CG to a piece ----
  u32x4 av[AD][MB][AQ];
  // a piece: staged, then the next one's loads sent off, and the first fragments read
  auto start_piece = [&](int ch) {
    stage_store();
    __syncthreads();
    if (!ONE && ch + CG < nc) stage_load(ch + CG);
#pragma unroll
    for (int d = 0; d < AD; ++d)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) frag_read(mb, d, 0, av[d][mb]);
  };
  if constexpr (ONE) start_piece(0);
#pragma unroll 1
  for (int ch = 0; ch < nc; ++ch) {
    const int sub = ch % CG;
    if constexpr (!ONE) {
      if (sub == 0) start_piece(ch);
    }
    // (past the last chunk: its first steps again, unused)
    const bool round_end = MULTI && (ch + 1) % pc == 0;
    const uint32_t wnext = ch + 1 < nc ? wbase + (round_end ? 3 * pc + 1 : 1) * S::CSTEP * wstep : wbase;
#pragma unroll
    for (int s = 0; s < NSTEP; ++s) {
      const int t = s + RING - 1;
      if (!ONE || CG > 1 || t < NSTEP) wload(t < NSTEP ? wbase + t * wstep : wnext + (t - NSTEP) * wstep, bq[t % RING]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = mfma(bq[s % RING][nb], av[s % AD][mb], acc[mb][nb]);
        if (s + AD < NSTEP)
          frag_read(mb, s + AD, 0, av[s % AD][mb]);
        else if (CG > 1 && sub + 1 < CG)  // (uniform) on into the piece's next chunk
          frag_read(mb, s + AD - NSTEP, 32, av[s % AD][mb]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    wbase = wnext;
    if constexpr (CG > 1) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) rbase[mb] += sub + 1 < CG ? 32u : (uint32_t)-(32 * (CG - 1));
    }
    if (sub == CG - 1) __syncthreads();  // every wave is done reading the staged piece
    if constexpr (MULTI) {
      if (round_end && ch + 1 < nc) {  // uniform: this round's sums are complete
        put_sums();
        __syncthreads();
#pragma unroll
        for (int ps = 0; ps < PASSES; ++ps) get_sums(ps, ch + 1 == pc, tot[ps]);
        __syncthreads();  // read before the next piece is staged over them
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mb][nb][v] = 0.0f;
      }
    }
  }
  put_sums();
  __syncthreads();

  // ---- epilogue: a lane finishes 8 channels of a row ----
  const int co = cg * TC + grp * 8;
  float bv[8], sv[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    bv[e] = consts[grp * 8 + e];
    if constexpr (F8) sv[e] = consts[TC + grp * 8 + e];
  }
  with_activation(p.act, [&](auto A) {
    constexpr int ACT = decltype(A)::value;
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) {
      const int r = (ps * 4 + wave) * RPW + lane / GPR;
      float v[8];
      if constexpr (MULTI) {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = tot[ps][e];
      }
      get_sums(ps, !MULTI, v);
      int a, c, e1;
      const bool ok = row_of(r, a, c, e1);
      const long long pidx = origin + mad24(a, p.P, mad24(c, p.Wp, e1)) - first + HW * (p.P + p.Wp + 1);
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = F8 ? __builtin_fmaf(v[e], sv[e], bv[e]) : v[e] + bv[e];
      if constexpr (EPI == 2) {
        // the output layer: channels 0..3 are the logits
        if (ok && grp == 0) {
          const int t = a0 + a, i = i0 + c, j = j0 + e1;
          const int HH = p.H * p.H, s = i * p.H + j;
          p.nib[(long long)b * p.g.V + (long long)t * HH + s] = (uint8_t)flip_nibble(p.g, p.tables, i, j, v);
          if (p.logits) {
#pragma unroll
            for (int o = 0; o < 4; ++o) p.logits[(((long long)b * 4 + o) * p.T + t) * HH + s] = v[o];
          }
        }
      } else if constexpr (EPI == 1) {
        // the 1x1x1 head on the rounded activations (the tile holds every channel of its voxels)
        float lg[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float h = F8 ? e4m3_round(act_fn<ACT>(v[e])) : bf16_round(act_fn<ACT>(v[e]));
#pragma unroll
          for (int o = 0; o < 4; ++o) lg[o] = __builtin_fmaf(consts[(2 + o) * TC + grp * 8 + e], h, lg[o]);
        }
#pragma unroll
        for (int m = GPR / 2; m >= 1; m >>= 1)
#pragma unroll
          for (int o = 0; o < 4; ++o) lg[o] += __shfl_xor(lg[o], m);
        if (ok && grp == 0) {
#pragma unroll
          for (int o = 0; o < 4; ++o) lg[o] += p.head_b[o];
          const int t = a0 + a, i = i0 + c, j = j0 + e1;
          const int HH = p.H * p.H, s = i * p.H + j;
          p.nib[(long long)b * p.g.V + (long long)t * HH + s] = (uint8_t)flip_nibble(p.g, p.tables, i, j, lg);
          if (p.logits) {
#pragma unroll
            for (int o = 0; o < 4; ++o) p.logits[(((long long)b * 4 + o) * p.T + t) * HH + s] = lg[o];
          }
        }
      } else if (ok) {
        if constexpr (EPI == 4) {  // the block's shortcut: its row, or its projection
          float sh[8];
          shortcut_of<8, F8>(p.sc, p.sc_stride, pidx, p.head_w, p.head_b, co, sh);
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] += sh[e];
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = act_fn<ACT>(v[e]);
        char* const out = p.y + (pidx * p.ystride + co) * ESZ;
        if constexpr (F8) {
          *reinterpret_cast<uint2*>(out) = uint2{e4m3_pack4(v[0], v[1], v[2], v[3]), e4m3_pack4(v[4], v[5], v[6], v[7])};
        } else {
          *reinterpret_cast<uint4*>(out) =
              uint4{bf16_pack(v[0], v[1]), bf16_pack(v[2], v[3]), bf16_pack(v[4], v[5]), bf16_pack(v[6], v[7])};
        }
      }
    }
  });
}

template <typename S, int EPI>
hipError_t launch(const SmallArgs& a, long long blocks, hipStream_t stream) {
  static std::atomic<uint64_t> done{0};
  const hipError_t e = allow_lds((const void*)conv_small_kernel<S, EPI>, S::lds, done);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((conv_small_kernel<S, EPI>), dim3((unsigned)blocks), dim3(NT), S::lds, stream, a);
  return hipGetLastError();
}

// Shape R x TC of P parts, if it is one of the instances.
template <int KS, bool F8, bool HALF, bool ONE, int KG, bool MULTI, int WM, int WN, int MB, int NB>
bool try_shape(const SmallArgs& a, long long blocks, const SmallPlan& pl, int epi, hipStream_t stream, hipError_t* e) {
  using S = Small<KS, F8, HALF, ONE, KG, MULTI, WM, WN, MB, NB>;
  const int kg = F8 ? 4 : std::min(pl.parts, 4);
  if (pl.rows != S::R || pl.cols != S::TC || kg != KG || (!F8 && (pl.parts > 4) != MULTI)) return false;
  if (epi == 0) {
    *e = launch<S, 0>(a, blocks, stream);
    return true;
  }
  if constexpr (KS == 3 && S::TC == 64 && S::R != 96) {  // (heads follow 64 or 128 input channels)
    if (epi == 1 && a.ncg == 1) {
      *e = launch<S, 1>(a, blocks, stream);
      return true;
    }
  }
  if constexpr (KS == 3 && S::TC <= 128) {
    if (epi == 4) {
      *e = launch<S, 4>(a, blocks, stream);
      return true;
    }
  }
  if constexpr (KS == 5 && S::TC == 32 && KG == 4 && !MULTI) {
    if (epi == 2) {
      *e = launch<S, 2>(a, blocks, stream);
      return true;
    }
  }
  return false;
}

template <int KS, bool ONE>
hipError_t launch_bf16(const SmallArgs& a, long long n, const SmallPlan& pl, int epi, hipStream_t st) {
  hipError_t e = hipErrorInvalidValue;
  // one part, two parts, four, more
  (void)(try_shape<KS, false, false, ONE, 1, false, 2, 2, 1, 1>(a, n, pl, epi, st, &e) ||
         try_shape<KS, false, false, ONE, 1, false, 2, 2, 2, 1>(a, n, pl, epi, st, &e) ||
         try_shape<KS, false, false, ONE, 1, false, 2, 2, 2, 2>(a, n, pl, epi, st, &e) ||
         try_shape<KS, false, false, ONE, 2, false, 2, 1, 1, 1>(a, n, pl, epi, st, &e) ||
         try_shape<KS, false, false, ONE, 2, false, 2, 1, 1, 2>(a, n, pl, epi, st, &e) ||
         try_shape<KS, false, false, ONE, 2, false, 2, 1, 2, 2>(a, n, pl, epi, st, &e) ||
         try_shape<KS, false, false, ONE, 4, false, 1, 1, 2, 1>(a, n, pl, epi, st, &e) ||
         try_shape<KS, false, false, ONE, 4, false, 1, 1, 2, 2>(a, n, pl, epi, st, &e) ||
         try_shape<KS, false, false, ONE, 4, false, 1, 1, 4, 1>(a, n, pl, epi, st, &e));
  if constexpr (!ONE) {
    if (e == hipErrorInvalidValue)
      (void)(try_shape<KS, false, false, ONE, 2, false, 1, 2, 3, 2>(a, n, pl, epi, st, &e) ||
             try_shape<KS, false, false, ONE, 4, true, 1, 1, 2, 1>(a, n, pl, epi, st, &e) ||
             try_shape<KS, false, false, ONE, 4, true, 1, 1, 2, 2>(a, n, pl, epi, st, &e));
  }
  if constexpr (!ONE && KS == 3) {
    if (e == hipErrorInvalidValue) (void)try_shape<KS, false, false, ONE, 4, false, 1, 1, 3, 2>(a, n, pl, epi, st, &e);
  }
  return e;
}

template <bool HALF, bool ONE>
hipError_t launch_fp8(const SmallArgs& a, long long n, const SmallPlan& pl, int epi, hipStream_t st) {
  hipError_t e = hipErrorInvalidValue;
  (void)(try_shape<3, true, HALF, ONE, 4, false, 1, 1, 2, 1>(a, n, pl, epi, st, &e) ||
         try_shape<3, true, HALF, ONE, 4, false, 1, 1, 2, 2>(a, n, pl, epi, st, &e) ||
         try_shape<3, true, HALF, ONE, 4, false, 1, 1, 4, 2>(a, n, pl, epi, st, &e));
  return e;
}

}  // namespace

hipError_t launch_conv_small(const SmallPlan& pl, const HiddenCall& c, bool fp8) {
  const Geom& g = *c.g;
  const Tiling& tl = *c.tl;
  const int cw = c.slice_width, row = c.cin * (fp8 ? 1 : 2), cols = pl.cols;
  const int cout = c.epi == 2 ? 32 : c.cout;  // the output layer's 4 filters fill one padded block
  if ((c.ks != 3 && c.ks != 5) || g.pad != (c.ks - 1) / 2 || tl.mode != 1 || tl.span <= 0 ||
      tl.span > conv_small_span(c.ks) || (c.ks == 5 && fp8))
    return hipErrorInvalidValue;
  if (cols <= 0 || cout % cols != 0 || cout % cw != 0 || cw % cols != 0 || (cw != 32 && cw != 64 && cw != 128))
    return hipErrorInvalidValue;
  if (row % 128 != 0 && !(fp8 && row == 64)) return hipErrorInvalidValue;
  if (c.epi == 4 && c.head_w && (!c.head_b || !c.sc || c.sc_stride < 1 || c.sc_stride > 8)) return hipErrorInvalidValue;
  // parts of whole chunks, of four a multiple past four
  const int nch = row / 32;
  if (!fp8 && (pl.parts < 1 ||  (pl.parts & (pl.parts - 1)) || nch % pl.parts))
    return hipErrorInvalidValue;
  SmallArgs a{};
  a.ncg = cout / cols;
  const long long blocks = tl.ntiles * a.ncg;
  if (blocks >= (1ll << 31)) return hipErrorInvalidValue;
  a.x = (const char*)c.x;
  a.wfrag = c.wfrag;
  a.y = (char*)c.y;
  a.bias = c.bias;
  a.head_w = c.head_w;
  a.head_b = c.head_b;
  a.sc = c.sc;
  a.S = g.S;
  a.xbytes = (long long)c.batch * g.S * row;
  a.T = g.T;
  a.H = g.H;
  a.Wp = g.Wp;
  a.P = g.P;
  a.BI = tl.BI;
  a.BJ = tl.BJ;
  a.sa = tl.sa;
  a.sb = tl.sb;
  a.span = tl.span;
  a.ntI = tl.ntI;
  a.ntJ = tl.ntJ;
  a.per = tl.ntT * tl.ntI * tl.ntJ;
  a.bij = tl.BI * tl.BJ;
  a.r_sa = 1.0f / (float)tl.sa;
  a.r_sb = 1.0f / (float)tl.sb;
  a.r_bij = 1.0f / (float)a.bij;
  a.r_bj = 1.0f / (float)tl.BJ;
  a.by_ncg = make_fastdiv((uint32_t)a.ncg);
  a.by_per = tl.dv_per;
  a.by_ij = tl.dv_ntij;
  a.by_j = tl.dv_ntj;
  a.by_bij = tl.dv_bij;
  a.by_bj = tl.dv_bj;
  a.act = c.act;
  a.row = row;
  a.np = row >= 128 ? row / 128 : 1;
  a.part_chunks = fp8 ? 0 : nch / pl.parts;
  a.ystride = c.ystride;
  a.nbt = cw / 32;
  a.lnbt = cw == 128 ? 2 : (cw == 64 ? 1 : 0);
  a.tsteps = fp8 ? c.cin / 32 * 14 : c.cin / 16 * c.ks * c.ks * c.ks;
  a.sc_stride = c.sc_stride;
  a.g = g;
  a.tables = c.tables;
  a.nib = c.nib;
  a.logits = c.logits;
  if (fp8) {
    if (row == 64) return launch_fp8<true, true>(a, blocks, pl, c.epi, c.stream);
    return a.np == 1 ? launch_fp8<false, true>(a, blocks, pl, c.epi, c.stream)
                     : launch_fp8<false, false>(a, blocks, pl, c.epi, c.stream);
  }
  if (c.ks == 5)
    return a.np == 1 ? launch_bf16<5, true>(a, blocks, pl, c.epi, c.stream)
                     : launch_bf16<5, false>(a, blocks, pl, c.epi, c.stream);
  return a.np == 1 ? launch_bf16<3, true>(a, blocks, pl, c.epi, c.stream)
                   : launch_bf16<3, false>(a, blocks, pl, c.epi, c.stream);
}

}  // namespace pd
