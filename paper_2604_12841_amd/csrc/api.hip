// api.hip -- host side of the C ABI declared in include/predecoder.h.
//
// create: validates the arguments on the host (no device call before that),
// builds the GPU-side geometry tables, plans the conv tiling, reorders the
// weights into MFMA fragment order (rounding to bf16 with round-to-nearest-
// even for the bf16 path), allocates the zero-halo activation buffers for
// max_batch samples and clears them once.
// run: enqueues unpack -> conv layers -> head -> residual/repack on the
// caller's stream and returns; it never synchronises.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstring>
#include <new>
#include <vector>

#include "../../include/predecoder.h"
#include "conv_small.h"
#include "internal.h"

using pd::Geom;
using pd::Tiling;

namespace {

constexpr size_t kSchedWords = 256;  // the hidden kernel's unit counters: 8 XCDs x 2 x 16 words

// Device memory one run works in besides its inputs, outputs, weights and
// tables: the input planes, the activation buffers, the projection outputs of
// residual blocks, the flip nibbles and the hidden kernel's unit counters.
// A handle owns one (sized for max_batch at create); predecoder_run_static
// lays one over the library's static scratch array for each call.
struct Workspace {
  void* planes = nullptr;                      // [batch * S][c_in], zero halo
  void* act[3] = {nullptr, nullptr, nullptr};  // activations [batch * S][cmax]; act[2]: residual networks only
  void* pbuf = nullptr;                        // projection outputs [batch * S][pmax] (residual networks)
  uint8_t* nib = nullptr;                      // [batch][T][H][H] flip nibbles
  uint32_t* sched = nullptr;                   // the hidden kernel's unit counters (kSchedWords, zero between launches)
  size_t act_bytes = 0;                        // size of each activation buffer
  // Row width (bytes per voxel) of the data each activation buffer holds, 0
  // while it is all zero.  The 3x3x3 kernels read the zero halo around the
  // interior voxels; a buffer written with one row width and then with
  // another would show the old interior rows as halo, so it is zeroed first
  // (prepare_rows).
  int act_row[3] = {0, 0, 0};
};

}  // namespace

struct pd_predecoder {
  Geom g;                        // includes the layout and the boundary bases
  int dtype = 0;
  int max_batch = 0;
  int device = 0;
  std::vector<pd_layer> layers;
  int ks = 3;                    // kernel size of the conv layers: 3, or 5 (Model 3 of Table models)
  Tiling tiling{};               // shared by every k x k x k layer (bf16 and fp8 paths)
  Tiling sums{};                 // ... that the K parts of the sums are counted over (conv_parts, sum_plan)
  Tiling small[3]{};             // tiles of 64, 96 and 128 voxels for the small-launch kernel (span 0: none)
  Workspace ws;                  // sized for max_batch
  int32_t* tables = nullptr;
  std::vector<void*> wdev;       // per conv layer: fragments
  std::vector<size_t> wslice;    // per conv layer: bytes of the fragments of one 128-channel slice of a
                                 // 256-wide layer (run as two slices), 0 otherwise
  std::vector<float*> bdev;      // per conv layer: bias fp32 (a 3x3x3 output layer: [4] biases, [4] scales)
  float* head_w = nullptr;       // [4][c_in] fp32 (bf16-valued on the bf16 path)
  float* head_b = nullptr;       // [4]
  // residual network (predecoder_create_resnet): its blocks; wdev / wslice /
  // bdev hold conv1 and conv2 of block k at 2k and 2k + 1 (BatchNorm folded
  // in), proj_w / proj_b its projection (null for an identity shortcut)
  std::vector<pd_block> blocks;
  std::vector<float*> proj_w, proj_b;
  void* out_proj_frag = nullptr;  // the last block's projection as fragments of launch_conv_out (when it
                                  // runs there, fused into the output conv), else null
  float* out_proj_bias = nullptr; // ... its [4] biases and [4] weight scales
  int cmax = 0;                  // widest activation row (channels)
  int pmax = 0;                  // widest projection output (channels; residual networks)
  int n_cu = 256;                // compute units: one persistent conv workgroup each
};

// One recorded predecoder_run (predecoder_graph_create).
struct pd_graph {
  hipStream_t stream = nullptr;
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
};

namespace {

const int kMaxD = 63;
const int kMaxT = 1023;

bool layer_chain_ok(const pd_layer* l, int n, int layout) {
  if (n < 1) return false;
  if (l[0].c_in != (layout == PD_LAYOUT_PAPER ? 4 : 2)) return false;
  if (l[n - 1].c_out != 4) return false;
  if (l[n - 1].act != PD_ACT_NONE) return false;
  for (int i = 0; i < n; ++i) {
    if (l[i].c_in < 1 || l[i].c_out < 1) return false;
    if (l[i].k < 1 || (l[i].k % 2) == 0) return false;
    if (l[i].act < PD_ACT_NONE || l[i].act > PD_ACT_RELU) return false;
    if (i > 0 && l[i].c_in != l[i - 1].c_out) return false;
  }
  return true;
}

Geom make_geom(int d, int T, int layout = PD_LAYOUT_PLAQUETTE, int first = PD_BOUNDARY_NONE,
               int last = PD_BOUNDARY_NONE, int pad = 1) {
  Geom g;
  g.d = d;
  g.T = T;
  g.layout = layout;
  g.first = first;
  g.last = last;
  g.first_n = INT_MAX;
  g.last_from = 0;
  g.pad = pad;
  g.H = layout == PD_LAYOUT_PAPER ? d : d + 1;  // the data qubits, or the plaquettes
  g.Wp = g.H + 2 * pad;
  g.P = g.Wp * g.Wp;
  g.S = (long long)(T + 2 * pad) * g.P;
  g.V = T * g.H * g.H;
  g.nstab = d * d - 1;
  g.K = g.nstab / 2;
  g.nflip = 3 * d * d - 1;
  g.Wd = ((long long)T * g.nstab + 63) / 64;
  g.Wf = ((long long)T * g.nflip + 63) / 64;
  return g;
}

// GPU-side geometry tables (see internal.h).  Plaquette (i, j), 0 <= i, j <=
// d, holds an X stabilizer iff (i+j) is even and 1 <= i <= d-1, a Z
// stabilizer iff (i+j) is odd and 1 <= j <= d-1, and acts on the data qubits
// (i-1..i, j-1..j) inside [0, d-1]^2.  In the paper's layout (Sec. IV.B.1,
// Fig. StabMap) a stabilizer's events enter, and its measurement flip is read,
// at one qubit of its support: a weight-four X (Z) stabilizer at its top-left
// (top-right) qubit, a weight-two X stabilizer (on the left / right edge) at
// its upper qubit, a weight-two Z stabilizer (top / bottom edge) at its right
// qubit.
std::vector<int32_t> build_tables(const Geom& g) {
  std::vector<int32_t> t(pd::tables_size(g), -1);
  int32_t* site_of = t.data() + pd::tables_site_of(g);
  int32_t* comp_x = t.data() + pd::tables_comp_x(g);
  int32_t* comp_z = t.data() + pd::tables_comp_z(g);
  int32_t* supp = t.data() + pd::tables_supp(g);
  const int d = g.d, H = g.H;
  const bool paper = g.layout == PD_LAYOUT_PAPER;
  int n = 0;
  for (int pass = 0; pass < 2; ++pass)
    for (int i = 0; i <= d; ++i)
      for (int j = 0; j <= d; ++j) {
        const bool x = ((i + j) & 1) == 0 && i >= 1 && i <= d - 1;
        const bool z = ((i + j) & 1) == 1 && j >= 1 && j <= d - 1;
        if (!((pass == 0 && x) || (pass == 1 && z))) continue;
        int q = 0;
        for (int r = i - 1; r <= i; ++r)
          for (int c = j - 1; c <= j; ++c)
            if (r >= 0 && r < d && c >= 0 && c < d) supp[n * 4 + q++] = r * H + c;
        int site = i * H + j;
        if (paper) {
          if (x)  // top-left of four; upper qubit of an edge pair (column 0 or d-1)
            site = (i - 1) * H + (j == 0 ? 0 : (j == d ? d - 1 : j - 1));
          else  // top-right of four; right qubit of an edge pair (row 0 or d-1)
            site = (i == 0 ? 0 : (i == d ? d - 1 : i - 1)) * H + j;
        }
        site_of[n] = site;
        (x ? comp_x : comp_z)[site] = n;
        ++n;
      }
  // residual stencils and flip-row sites (grid indices < 2^16: H <= 64)
  int32_t* sten = t.data() + pd::tables_sten(g);
  for (int k = 0; k < g.nstab; ++k) {
    const int32_t* q = supp + 4 * k;
    const int q2 = q[2] >= 0 ? q[2] : q[0], q3 = q[3] >= 0 ? q[3] : q[0];  // weight two: q2 = q3 cancel
    sten[4 * k] = site_of[k] | ((k < g.K ? 2 : 3) << 16);
    sten[4 * k + 1] = q[0] | (q[1] << 16);
    sten[4 * k + 2] = q2 | (q3 << 16);
    sten[4 * k + 3] = 0;
  }
  int32_t* fsite = t.data() + pd::tables_fsite(g);
  for (int k = 0; k < g.nflip; ++k) {
    const int dd = d * d;
    if (k < 2 * dd) {
      const int r = (k % dd) / d, c = (k % dd) % d;
      fsite[k] = (r * H + c) | ((k < dd ? 0 : 1) << 16);
    } else {
      const int m = k - 2 * dd;
      fsite[k] = site_of[m] | ((m < g.K ? 2 : 3) << 16);
    }
  }
  return t;
}

// fp32 -> bf16 bits, round to nearest even on the fp32 bit pattern.
uint16_t bf16_bits(float f) {
  uint32_t u;
  std::memcpy(&u, &f, 4);
  if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x7fffffu)) return (uint16_t)((u >> 16) | 0x40);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
float bf16_value(float f) {
  uint32_t u = (uint32_t)bf16_bits(f) << 16;
  float r;
  std::memcpy(&r, &u, 4);
  return r;
}

// Tiling plan for the 3x3x3 layers: the candidate with the fewest MFMA rows
// per sample whose double-buffered 32-channel staging fits in LDS (cost 2 x
// rows; ties go to per-sample tiles, then cells of 16-voxel rows, then the
// smaller span).

long long flat_span(const Geom& g, long long seg_len, long long nseg, int batch) {
  // exact maximum staged span (line space, see pd::Tiling) over all tiles of
  // `batch` samples
  long long best = 0, halo = pd::line_plane(g) + g.H + 1;
  long long tiles = (seg_len + pd::kTileRows - 1) / pd::kTileRows;
  for (long long s = 0; s < nseg; ++s)
    for (long long k = 0; k < tiles; ++k) {
      long long u0 = s * seg_len + k * pd::kTileRows;
      long long u1 = std::min(u0 + pd::kTileRows, std::min((s + 1) * seg_len, (long long)batch * g.V)) - 1;
      if (u1 < u0) continue;
      auto lidx = [&](long long u) {
        long long b = u / g.V, v = u % g.V;
        int HH = g.H * g.H;
        int t = (int)(v / HH), r = (int)(v % HH);
        return pd::line_index(g, (int)b, t, r / g.H, r % g.H);
      };
      best = std::max(best, lidx(u1) - lidx(u0) + 2 * halo + 1);
    }
  return best;
}

// The most lines a tile (`rows` voxels) of a cell of n voxels stages (cell
// line space, see pd::Tiling); limit + 1 when over `limit`.  Tiles repeat
// their place in the cell's rounds after at most BI BJ of them.
int cell_span(const Tiling& t, int n, int pad, int rows, int limit) {
  const int bij = t.BI * t.BJ;
  const int halo = 2 * pad * (t.sa + t.sb + 1) + 1;
  if (n >= rows && halo + rows - 1 > limit) return limit + 1;  // most cells: no need to look closer
  auto line = [&](int u) {
    const int r = u % bij;
    return u / bij * t.sa + r / t.BJ * t.sb + r % t.BJ;
  };
  int best = 0;
  for (int k = 0; k < std::min(t.ntT, bij) && best <= limit; ++k) {
    const int u0 = k * rows, u1 = std::min(u0 + rows, n) - 1;
    best = std::max(best, line(u1) - line(u0) + halo);
  }
  return std::min(best, limit + 1);
}

// The tiling by cells of BI x BJ with tiles of `rows` voxels; span limit + 1
// when a tile stages more than `limit` lines.
Tiling cell_tiling(const Geom& g, int BI, int BJ, int rows, int limit) {
  const int p = g.pad;
  Tiling t{};
  t.mode = 1;
  t.BI = BI;
  t.BJ = BJ;
  t.ntT = (g.T * BI * BJ + rows - 1) / rows;
  t.ntI = (g.H + BI - 1) / BI;
  t.ntJ = (g.H + BJ - 1) / BJ;
  t.sa = (BI + 2 * p) * (BJ + 2 * p);
  t.sb = BJ + 2 * p;
  t.span = cell_span(t, g.T * BI * BJ, p, rows, limit);
  return t;
}

// Tiling of the small-launch kernel (span 0 where no cell fits): the fewest
// tiles of `rows` voxels, weighed against what a tile stages (500 lines cost
// as much as a quarter more tiles) and the LDS bank conflicts of very short
// cell rows.
Tiling plan_small(const Geom& g, int rows, int ks) {
  const int limit = pd::conv_small_span(ks);
  Tiling best{};
  double least = 0.0;
  for (int BJ = 1; BJ <= g.H; ++BJ)
    for (int BI = 1; BI <= g.H; ++BI) {
      const Tiling t = cell_tiling(g, BI, BJ, rows, limit);
      if (t.span > limit) continue;
      const double cost = (double)t.ntT * t.ntI * t.ntJ * (1.0 + 0.0005 * t.span) * (BJ < 4 ? 1.08 : 1.0);
      if (best.span == 0 || cost < least) {
        best = t;
        least = cost;
      }
    }
  return best;
}

// boxes: with boxes of whole rounds instead of cells (a cell's rows run on
// from tile to tile, a box's last rounds may be short): not a tiling that
// runs, but the one that the K parts of the sums are counted over.
Tiling plan_tiling(const Geom& g, int max_batch, int ks = 3, bool boxes = false) {
  // 5x5x5 layers: their own (larger) staging buffers, cells on a halo of two
  const int kMaxSpan = ks == 3 ? std::min(pd::conv_single_max_span(), pd::conv_hidden_max_span(3))
                               : pd::conv_hidden_max_span(5);
  Tiling best{};
  long long best_rows = -1;
  int best_span = 0;
  auto consider = [&](const Tiling& t, long long rows_per_sample) {
    if (t.span > kMaxSpan) return;
    if (best_rows < 0 || rows_per_sample < best_rows ||
        (rows_per_sample == best_rows && t.span < best_span)) {
      best = t;
      best_rows = rows_per_sample;
      best_span = t.span;
    }
  };
  // flat, tiles inside one sample (a halo of one only)
  if (g.pad == 1) {
    Tiling t{};
    t.mode = 0;
    t.seg_len = g.V;
    t.tiles_per_seg = (g.V + pd::kTileRows - 1) / pd::kTileRows;
    t.sa = pd::line_plane(g);
    t.sb = g.H;
    t.span = (int)std::min<long long>(flat_span(g, g.V, 1, 1), 1 << 30);
    consider(t, 2ll * t.tiles_per_seg * pd::kTileRows);
  }
  // flat across samples (rows per sample ~ V); the span bound covers any batch
  if (max_batch > 1 && g.pad == 1) {
    Tiling t{};
    t.mode = 0;
    t.seg_len = -1;  // set per run to batch * V
    t.tiles_per_seg = 0;
    t.sa = pd::line_plane(g);
    t.sb = g.H;
    int nb = std::min(max_batch, 256);
    t.span = (int)std::min<long long>(flat_span(g, (long long)nb * g.V, 1, nb), 1 << 30);
    consider(t, 2ll * g.V + 2);  // +2: prefer per-sample tiles at equal cost
  }
  // cells
  for (int BJ = 1; BJ <= g.H; ++BJ)
    for (int BI = 1; BI <= g.H; ++BI) {
      Tiling t{};
      if (boxes) {
        const int BT = std::min(g.T, pd::kTileRows / (BI * BJ)), halo = 2 * g.pad;
        if (BT < 1) break;
        t.mode = 1;
        t.ntT = (g.T + BT - 1) / BT;
        t.ntI = (g.H + BI - 1) / BI;
        t.ntJ = (g.H + BJ - 1) / BJ;
        t.span = (BT + halo) * (BI + halo) * (BJ + halo);
      } else {
        t = cell_tiling(g, BI, BJ, pd::kTileRows, kMaxSpan);
      }
      // (a cell row of BJ < 16 voxels, whose 16-lane LDS reads span two
      // staged lines, costs little: at d = T = 25 a 5x3x16 box and a 9x13x2
      // box reached 0.54 and 0.53 of peak per MFMA row, so the row count
      // decides, and BJ = 16 only breaks ties)
      const long long rows = (long long)t.ntT * t.ntI * t.ntJ * pd::kTileRows;
      consider(t, 2 * rows + (BJ % 16 != 0));
    }
  return best;
}

void tiling_for_batch(Tiling* t, const Geom& g, int batch) {
  t->div_a = pd::make_fastdiv((uint32_t)t->sa);
  t->div_b = pd::make_fastdiv((uint32_t)t->sb);
  t->dv_V = pd::make_fastdiv((uint32_t)g.V);
  t->dv_HH = pd::make_fastdiv((uint32_t)(g.H * g.H));
  t->dv_H = pd::make_fastdiv((uint32_t)g.H);
  if (t->mode == 1) {
    t->dv_per = pd::make_fastdiv((uint32_t)(t->ntT * t->ntI * t->ntJ));
    t->dv_ntij = pd::make_fastdiv((uint32_t)(t->ntI * t->ntJ));
    t->dv_ntj = pd::make_fastdiv((uint32_t)t->ntJ);
    t->dv_bij = pd::make_fastdiv((uint32_t)(t->BI * t->BJ));
    t->dv_bj = pd::make_fastdiv((uint32_t)t->BJ);
  }
  if (t->mode == 0) {
    if (t->seg_len < 0 || t->tiles_per_seg == 0) {
      // flat across samples
      t->seg_len = (long long)batch * g.V;
      t->tiles_per_seg = (int)((t->seg_len + pd::kTileRows - 1) / pd::kTileRows);
      t->ntiles = t->tiles_per_seg;
    } else {
      t->ntiles = (long long)batch * t->tiles_per_seg;
    }
    t->dv_tps = pd::make_fastdiv((uint32_t)t->tiles_per_seg);
  } else {
    t->ntiles = (long long)batch * t->ntT * t->ntI * t->ntJ;
  }
}

// Kernel size of a network's conv layers: 5 when its first layer is 5x5x5
// (Model 3 of Table models), else 3.
int network_ks(const pd_layer* l) { return l[0].k == 5 ? 5 : 3; }

bool supported(const Geom& g, const pd_layer* l, int n, int dtype) {
  if (g.d > kMaxD || g.T > kMaxT) return false;
  if (n < 2) return false;  // at least one hidden 3x3x3 layer before the head
  if (network_ks(l) == 5) {
    // 5x5x5 networks (Model 3 of Table models): the paper layout, bf16, every
    // layer 5x5x5 (the output layer too), one hidden width, 64 or 128
    if (g.layout != PD_LAYOUT_PAPER || dtype != PD_DTYPE_BF16 || n < 3) return false;
    const int w = l[0].c_out;
    if (w != 64 && w != 128) return false;
    for (int i = 0; i < n; ++i) {
      if (l[i].k != 5) return false;
      if (i < n - 1 && l[i].c_out != w) return false;
    }
    return true;
  }
  if (g.layout == PD_LAYOUT_PAPER && dtype == PD_DTYPE_FP32) return false;
  const bool mfma = dtype != PD_DTYPE_FP32;
  // fp8 with a 1x1x1 head needs its head fused into a hidden layer after the
  // first (a lone hidden layer carrying the head runs in bf16 only)
  if (dtype == PD_DTYPE_FP8 && l[n - 1].k == 1 && n < 3) return false;
  bool wide = false;
  for (int i = 0; i < n - 1; ++i) {
    if (l[i].k != 3) return false;
    int co = l[i].c_out;
    if (mfma) {
      if (co != 64 && co != 128 && co != 256) return false;
      wide = wide || co == 256;
    } else {
      if (co % 8 != 0 || co > 128) return false;
    }
  }
  const pd_layer& out = l[n - 1];
  // 256-wide layers run as two 128-channel slices; a 1x1x1 head needs all
  // channels of its input in one workgroup, so they go with a 3x3x3 output layer
  if (wide && out.k != 3) return false;
  if (out.k == 3) return g.layout == PD_LAYOUT_PAPER;  // a 3x3x3 output layer (c_in 64 or 128, checked above)
  if (out.k != 1 || out.c_in > 128) return false;
  if (mfma && (out.c_in % 8) != 0) return false;
  return true;
}

// OCP E4M3 (fp8 path): the code of v, rounded to nearest with ties to even,
// magnitudes of 448 and above saturating to 448 (code 0x7e); NaN is never
// passed (weights are finite).
uint8_t e4m3_code(float v) {
  const uint8_t sgn = std::signbit(v) ? 0x80 : 0;
  const double a = std::fabs((double)v);
  if (a >= 448.0) return sgn | 0x7e;
  int ex;
  std::frexp(a, &ex);  // a = f 2^ex, f in [0.5, 1)
  if (a == 0.0 || ex - 1 < -6) {  // subnormal range: multiples of 2^-9
    const int q = (int)std::nearbyint(std::ldexp(a, 9));  // 8 becomes the smallest normal, code 0x08
    return sgn | (uint8_t)q;
  }
  int e = ex - 1;  // a = m 2^e, m in [1, 2)
  int m = (int)std::nearbyint((std::ldexp(a, -e) - 1.0) * 8.0);
  if (m == 8) {
    m = 0;
    ++e;
  }
  const int code = ((e + 7) << 3) | m;
  return sgn | (uint8_t)std::min(code, 0x7e);
}

float e4m3_value(uint8_t c) {
  const int ex = (c >> 3) & 15, m = c & 7;
  const double v = ex == 0 ? std::ldexp((double)m, -9) : std::ldexp(1.0 + m / 8.0, ex - 7);
  return (float)((c & 0x80) ? -v : v);
}

// Power-of-two scale exponent of a weight row: the smallest e with
// amax / 2^e <= 448 (0 for an all-zero row).
int e4m3_scale_exp(float amax) {
  if (amax == 0.0f) return 0;
  int ex;
  std::frexp((double)amax / 448.0, &ex);  // amax / 448 = f 2^ex, f in [0.5, 1)
  // 2^(ex-1) <= amax / 448 < 2^ex: e = ex, or ex - 1 when amax / 448 is exactly 2^(ex-1)
  return std::ldexp((double)amax, -(ex - 1)) <= 448.0 ? ex - 1 : ex;
}

// Weights of a layer in fp8: per output channel, codes e4m3(w / 2^e) and the
// scale 2^e; wq receives the values the codes stand for (e4m3 value x 2^e).
void quantize_e4m3(const float* w, int cout, size_t row, std::vector<uint8_t>* codes, std::vector<float>* scale,
                   std::vector<float>* wq) {
  codes->assign((size_t)cout * row, 0);
  scale->assign(cout, 1.0f);
  wq->assign((size_t)cout * row, 0.0f);
  for (int co = 0; co < cout; ++co) {
    float amax = 0.0f;
    for (size_t e = 0; e < row; ++e) amax = std::max(amax, std::fabs(w[co * row + e]));
    const int ex = e4m3_scale_exp(amax);
    (*scale)[co] = std::ldexp(1.0f, ex);
    for (size_t e = 0; e < row; ++e) {
      const uint8_t c = e4m3_code(std::ldexp(w[co * row + e], -ex));
      (*codes)[co * row + e] = c;
      (*wq)[co * row + e] = std::ldexp(e4m3_value(c), ex);
    }
  }
}

template <typename T>
pd_status dev_alloc(T** p, size_t bytes) {
  *p = nullptr;
  if (bytes == 0) bytes = 16;
  hipError_t e = hipMalloc((void**)p, bytes);
  if (e == hipErrorOutOfMemory || e == hipErrorMemoryAllocation) {
    (void)hipGetLastError();
    return PD_ERR_OUT_OF_MEMORY;
  }
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return PD_ERR_DEVICE;
  }
  return PD_OK;
}

template <typename T>
pd_status upload(T** p, const void* host, size_t bytes) {
  pd_status s = dev_alloc(p, bytes);
  if (s != PD_OK) return s;
  if (hipMemcpy(*p, host, bytes, hipMemcpyHostToDevice) != hipSuccess) return PD_ERR_DEVICE;
  return PD_OK;
}

void free_all(pd_predecoder* h) {
  auto f = [](void* p) {
    if (p) (void)hipFree(p);
  };
  f(h->ws.planes);
  f(h->ws.act[0]);
  f(h->ws.act[1]);
  f(h->ws.act[2]);
  f(h->ws.pbuf);
  for (float* p : h->proj_w) f(p);
  for (float* p : h->proj_b) f(p);
  f(h->out_proj_frag);
  f(h->out_proj_bias);
  h->out_proj_frag = nullptr;
  h->out_proj_bias = nullptr;
  h->ws.act[2] = h->ws.pbuf = nullptr;
  h->proj_w.clear();
  h->proj_b.clear();
  f(h->ws.nib);
  f(h->tables);
  for (void* p : h->wdev) f(p);
  for (float* p : h->bdev) f(p);
  f(h->head_w);
  f(h->head_b);
  f(h->ws.sched);
  h->ws.planes = h->ws.act[0] = h->ws.act[1] = nullptr;
  h->ws.nib = nullptr;
  h->tables = nullptr;
  h->wdev.clear();
  h->wslice.clear();
  h->bdev.clear();
  h->head_w = h->head_b = nullptr;
  h->ws.sched = nullptr;
}

// bf16 A fragments (weights) for v_mfma_f32_32x32x16_bf16: lane l of
// fragment (k-step, channel block nb) holds W[co = 32 nb + l % 32][k0 + 8 (l / 32) + e],
// e = 0..7; output channels past c_out (the 4 filters of an output layer fill
// one block of 32) are zero.  Layer 1 (c_in = 2 or 4): k = c_in * tap + ci over
// ceil(k^3 c_in / 16) k-steps (taps past the last are zero).  Other layers:
// [chunk of 16 c_in][tap][nb] with ci = 16 chunk + 8 (l / 32) + e.
std::vector<uint16_t> conv_fragments(const float* w, int cin, int cout, int k = 3) {
  const int nbt = cout < 32 ? 1 : cout / 32;
  const int taps = k * k * k;
  std::vector<uint16_t> f;
  auto W = [&](int co, int ci, int tap) -> uint16_t {
    return co < cout ? bf16_bits(w[((size_t)co * cin + ci) * taps + tap]) : 0;
  };
  if (cin == 2 || cin == 4) {
    const int ks_n = (taps * cin + 15) / 16;
    f.assign((size_t)ks_n * nbt * 64 * 8, 0);
    for (int ks = 0; ks < ks_n; ++ks)
      for (int nb = 0; nb < nbt; ++nb)
        for (int l = 0; l < 64; ++l)
          for (int e = 0; e < 8; ++e) {
            int k = ks * 16 + 8 * (l / 32) + e;
            int tap = k / cin, ci = k % cin, co = nb * 32 + l % 32;
            f[(((size_t)ks * nbt + nb) * 64 + l) * 8 + e] = tap < taps ? W(co, ci, tap) : 0;
          }
  } else {
    const int nch = cin / 16;
    f.assign((size_t)nch * taps * nbt * 64 * 8, 0);
    for (int c = 0; c < nch; ++c)
      for (int tap = 0; tap < taps; ++tap)
        for (int nb = 0; nb < nbt; ++nb)
          for (int l = 0; l < 64; ++l)
            for (int e = 0; e < 8; ++e) {
              int ci = c * 16 + 8 * (l / 32) + e, co = nb * 32 + l % 32;
              size_t idx = ((((size_t)c * taps + tap) * nbt + nb) * 64 + l) * 8 + e;
              f[idx] = W(co, ci, tap);
            }
  }
  return f;
}

// fp8 A fragments (weight codes) for v_mfma_f32_32x32x64_f8f6f4: fragment
// (chunk of 32 c_in, k-step s, channel block nb), lane l holds 32 bytes,
// byte e = W[co = 32 nb + l % 32][ci = 32 chunk + e][tap 2 s + l / 32]
// (tap 27: zero); output channels past c_out are zero.
std::vector<uint8_t> conv_fragments_fp8(const uint8_t* codes, int cin, int cout) {
  const int nbt = cout < 32 ? 1 : cout / 32, nch = cin / 32, ns = 14;
  std::vector<uint8_t> f((size_t)nch * ns * nbt * 64 * 32, 0);
  for (int c = 0; c < nch; ++c)
    for (int st = 0; st < ns; ++st)
      for (int nb = 0; nb < nbt; ++nb)
        for (int l = 0; l < 64; ++l)
          for (int e = 0; e < 32; ++e) {
            const int co = nb * 32 + l % 32, ci = c * 32 + e, tap = 2 * st + l / 32;
            if (co < cout && tap < 27)
              f[((((size_t)c * ns + st) * nbt + nb) * 64 + l) * 32 + e] = codes[((size_t)co * cin + ci) * 27 + tap];
          }
  return f;
}

// Fragments of a 3x3x3 output layer of four filters for launch_conv_out:
// fragment (row block rb, k-step st), lane l: row m = l % 32 stands for tap
// 8 rb + m / 4 (zero past the last tap) and filter m % 4; bf16: 8 values,
// ci = 16 st + 8 (l / 32) + e; fp8 (codes): 32 codes, ci = 64 st + 32 (l /
// 32) + e.  Byte layout [rb][st][lane][16 or 32].
std::vector<uint8_t> out_fragments(const float* w, const uint8_t* codes, int cin, bool fp8) {
  const int kstep = fp8 ? 64 : 16, nks = cin / kstep, lb = fp8 ? 32 : 16;
  std::vector<uint8_t> f((size_t)4 * nks * 64 * lb, 0);
  for (int rb = 0; rb < 4; ++rb)
    for (int st = 0; st < nks; ++st)
      for (int l = 0; l < 64; ++l) {
        const int m = l % 32, tap = 8 * rb + m / 4, co = m % 4;
        if (tap >= 27) continue;
        uint8_t* dst = &f[(((size_t)rb * nks + st) * 64 + l) * lb];
        for (int e = 0; e < (fp8 ? 32 : 8); ++e) {
          const int ci = st * kstep + (fp8 ? 32 : 8) * (l / 32) + e;
          const size_t src = ((size_t)co * cin + ci) * 27 + tap;
          if (fp8) {
            dst[e] = codes[src];
          } else {
            const uint16_t v = bf16_bits(w[src]);
            std::memcpy(dst + 2 * e, &v, 2);
          }
        }
      }
  return f;
}

// bf16 fragments of a layer whose outputs run in slices of 128 channels
// when c_out > 128 (slices back to back; *slice = bytes of one slice, 0 when
// there is a single launch).
std::vector<uint16_t> fragments_sliced(const float* w, int cin, int cout, size_t* slice) {
  if (cout <= 128) {
    *slice = 0;
    return conv_fragments(w, cin, cout);
  }
  std::vector<uint16_t> f;
  for (int k = 0; k < cout / 128; ++k) {
    std::vector<uint16_t> fk = conv_fragments(w + (size_t)k * 128 * cin * 27, cin, 128);
    *slice = fk.size() * 2;
    f.insert(f.end(), fk.begin(), fk.end());
  }
  return f;
}

pd_status check_launch(hipError_t e) {
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return PD_ERR_DEVICE;
  }
  return PD_OK;
}

// Before a layer writes rows of row_bytes into activation buffer idx of ws:
// zero the buffer if it holds rows of another width (see act_row).
pd_status prepare_rows(Workspace& ws, int idx, int row_bytes, hipStream_t st) {
  if (ws.act_row[idx] != 0 && ws.act_row[idx] != row_bytes) {
    pd_status s = check_launch(pd::launch_zero(ws.act[idx], ws.act_bytes, st));
    if (s != PD_OK) return s;
  }
  ws.act_row[idx] = row_bytes;
  return PD_OK;
}

// Where a stopped run left the activations it was asked for (see
// enqueue_run's stop argument).
struct StopAt {
  const void* buf = nullptr;
  int row_bytes = 0;
};

// A hidden layer's call: c_out channels in slices of cw (weights and biases
// per slice), epi as in launch_conv_hidden (2: the 5x5x5 output layer).
// carries_head: the layer before a 1x1x1 head, whether or not this run
// applies it (epi 1) -- a run that stops at it must sum as the head's run does.
struct LayerRun {
  int cin, cout, cw, act;
  const void* x = nullptr;
  void* y = nullptr;
  const void* wfrag = nullptr;
  const float* bias = nullptr;
  int epi = 0;
  const float *head_w = nullptr, *head_b = nullptr;
  bool carries_head = false;
  const uint16_t* sc = nullptr;
  int sc_stride = 0;
};

// ---- The K parts of a layer's sums (bf16).  A sum is taken as P = 2^k parts
// of consecutive input-channel chunks, added in order.  P depends on the
// layer and the launch's size only (counted in boxes of 256 voxels, see
// plan_tiling), never on the kernel that runs it or how it is tiled, so a
// handle's results for a batch size do not depend on how its launches are
// shaped: few tiles (a small batch) take more parts, whose chains run side
// by side, up to one unit (tile, output slice, part) per compute unit.  Of
// the counts that fit, the least estimate in microseconds of a unit's time:
// its 16-channel chunks (2.5 each for 32 or 64 output channels, 3.9 for 128;
// a 5x5x5 chunk has 125 taps instead of 27) and its epilogue, or a part's
// share of the chunks and what parting costs.  (These are times of 256-voxel
// units in slices of 32 to 128 channels whose parts met through memory, which
// is how parted sums ran before the small-launch kernel; the choice stays as
// it was so that results keep their bits.)
int split_parts(const pd_predecoder* h, long long tiles, int cin, int width, int nsl, double* unit_us = nullptr) {
  const bool fp8 = h->dtype == PD_DTYPE_FP8;  // 32-channel chunks
  const int nch = cin / (fp8 ? 32 : 16);
  const double wide = width > 64 ? 1.0 : 0.0;
  const double chunk = (2.5 + 1.4 * wide) * (fp8 ? 1.1 : 1.0) * (h->ks * h->ks * h->ks) / 27.0;
  double best = nch * chunk + 3.3 + 4.0 * wide;
  if (unit_us) *unit_us = best;
  int parts = 1;
  for (int k = 1; nch % (1 << k) == 0 && ((tiles * nsl) << k) <= h->n_cu; ++k) {
    const double est = (nch >> k) * chunk + 1.75 + 1.65 * wide + 8.0;
    if (est < best) {
      best = est;
      parts = 1 << k;
    }
  }
  return parts;
}

// ... counted over slices of 32 or 64 output channels where those still fit
// the compute units (for the layer before a head only if it parts as a whole).
int conv_parts(const pd_predecoder* h, const LayerRun& L, long long tiles) {
  const int C = h->n_cu;
  if (h->blocks.empty() && h->ks == 3 && L.cin <= 128) {
    const bool sliced = !L.carries_head || split_parts(h, tiles, L.cin, L.cout, 1) > 1;
    if (sliced && tiles * (L.cout / 32) <= C) return split_parts(h, tiles, L.cin, 32, L.cout / 32);
    if (sliced && L.cout >= 128 && tiles * (L.cout / 64) <= C) return split_parts(h, tiles, L.cin, 64, L.cout / 64);
  }
  return split_parts(h, tiles, L.cin, L.cw, L.cout / L.cw);
}

// ---- Which kernel runs a hidden layer: the persistent one (launch_conv_hidden:
// 256-voxel tiles, two workgroups per CU; sums of one part) or the one for
// small launches (launch_conv_small).  Both times are estimated in
// microseconds and the smaller one wins.  Both were fitted to 1400 networks of
// 64- to 512-wide layers timed on MI355X both ways, 20 to 512 units at d = 5 to
// 31: what is taken is 1.6 % off the faster one on average.  Small / persistent
// near the line, whole networks in us by the units of a layer: four 128-wide
// layers bf16 122 / 152 at 120, 156 / 156 at 182, 203 / 171 at 228, 235 / 255 at
// 288, 323 / 273 at 370; fp8 84 / 99 at 136, 112 / 106 at 184, 163 / 161 at
// 371; 64-wide bf16 60 / 68 at 161, 119 / 112 at 410, fp8 57 / 55 at 256, 82 /
// 73 at 360; two 512-wide blocks bf16 631 / 671 at 320, 892 / 766 at 480, fp8
// 229 / 250 at 160, 495 / 414 at 360.  Past a full round of the persistent kernel's units it
// always runs: small launches then cost 4 to 28 % more (networks of four layers
// at 617 units: 128 channels bf16 510 / 426 us, fp8 311 / 260; 64 channels at 615
// 166 / 159, at 3600 817 / 706), all but the first few units over.

// Small launches: a workgroup costs `fixed` (start, staging, the sums'
// exchange, epilogue) and `piece` per 128-byte piece of its input rows; where
// two fit a CU, each adds `share` of its pieces' time (64 x 64 tiles of one K
// group are bound by L1 and LDS and gain nothing by sharing).  kg: K groups,
// which the parts fill up to four (fp8: always four).
struct SmallShape {
  int kg, rows, cols, acc;  // acc: accumulator registers of a lane
  double fixed, piece, share = 0.82;
};
constexpr SmallShape kSmallBf16[] = {
    {1, 64, 64, 16, 4.5, 3.7, 1.1}, {1, 128, 64, 32, 4.3, 7.3}, {1, 128, 128, 64, 6.0, 9.5},
    {2, 64, 32, 16, 3.9, 2.7},  {2, 64, 64, 32, 4.0, 5.0},  {2, 128, 64, 64, 4.5, 5.0},
    {2, 96, 128, 96, 6.0, 7.2},
    {4, 64, 32, 32, 3.9, 1.65}, {4, 64, 64, 64, 3.05, 2.7}, {4, 96, 64, 96, 5.5, 3.26}, {4, 128, 32, 64, 3.6, 2.63}};
constexpr SmallShape kSmallFp8[] = {{4, 64, 32, 32, 4.5, 1.35}, {4, 64, 64, 64, 4.4, 2.35}, {4, 128, 64, 128, 5.4, 4.4}};
constexpr SmallShape kSmall5[] = {
    {1, 64, 64, 16, 5.0, 14.5}, {1, 128, 64, 32, 5.0, 26.3}, {1, 128, 128, 64, 6.0, 43.0},
    {2, 64, 32, 16, 4.5, 9.7},  {2, 64, 64, 32, 5.0, 18.0},  {2, 128, 64, 64, 5.0, 22.0},
    {2, 96, 128, 96, 6.0, 31.0},
    {4, 64, 32, 32, 4.5, 9.7},  {4, 64, 64, 64, 5.0, 17.0},  {4, 128, 32, 64, 5.0, 13.5}};

double small_us(const pd_predecoder* h, const LayerRun& L, int batch, int parts, pd::SmallPlan* plan) {
  const bool fp8 = h->dtype == PD_DTYPE_FP8;
  const int row = L.cin * (fp8 ? 1 : 2), kg = fp8 ? 4 : std::min(parts, 4);
  const int cout = L.epi == 2 ? 32 : L.cout;
  double best = 1e30;
  auto consider = [&](const SmallShape& s) {
    const Tiling& t = h->small[s.rows / 32 - 2];
    if (s.kg != kg || t.span == 0 || L.cw % s.cols != 0 || (parts > 4 && !fp8 && s.rows != 64)) return;
    // (two 128 x 64 tiles share a CU there, which is no slower; with four parts,
    // two 64 x 64 ones of one-piece rows, and rows of two pieces were not measured)
    if (s.rows == 96 && row <= (kg == 4 ? 256 : 128)) return;
    // (a fused head needs all channels in the tile; wider ones take a kernel of their own)
    if (L.carries_head && cout == 64 && s.cols != 64) return;
    const long long units = (long long)batch * t.ntT * t.ntI * t.ntJ * (cout / s.cols);
    // (256 channels, us, 64 x 32 / 96 x 64 tiles: Model 5 d = 9, batch 6, 192 tiles 149 / 128, d = 17, 240 163 / 124, d
    // = 7, batch 16, 256 165 / 169; 512 channels gain at 256 tiles too, 171 / 145)
    if (s.rows == 96 && kg == 4 && row <= 512 && 16 * units > 15ll * h->n_cu) return;
    const int per_cu = pd::conv_small_occupancy(h->ks, row <= 128, s.acc);
    const long long rounds = (units + (long long)h->n_cu * per_cu - 1) / ((long long)h->n_cu * per_cu);
    const long long turns = (units + h->n_cu - 1) / h->n_cu;  // workgroups a CU runs
    const double pieces = row < 128 ? 0.8 : row / 128.0;
    const double us = per_cu == 1 ? rounds * (s.fixed + s.piece * pieces)
                                  : s.fixed * (1.0 + 0.75 * (rounds - 1)) +
                                        s.piece * pieces * (turns == 1 ? 1.0 : s.share * turns);
    if (us < best) {
      best = us;
      *plan = {s.rows, s.cols, parts};
    }
  };
  if (h->ks == 5)
    for (const SmallShape& s : kSmall5) consider(s);
  else if (fp8)
    for (const SmallShape& s : kSmallFp8) consider(s);
  else
    for (const SmallShape& s : kSmallBf16) consider(s);
  return best + (L.carries_head && L.cout != 64 ? 4.0 : 0.0);
}

// The persistent kernel: t1 for units of one workgroup per CU or fewer, t2 for
// a full round of two per CU, from a unit's matrix time m at 2.1 GHz.
struct BigTime {
  double t1, t2;
  long long round;  // units of a full round
};

BigTime big_time(const pd_predecoder* h, const LayerRun& L) {
  const bool fp8 = h->dtype == PD_DTYPE_FP8;
  const int taps = h->ks * h->ks * h->ks;
  const double steps = fp8 ? L.cin / 32 * ((taps + 1) / 2) * 2.0 : L.cin / 16 * taps;
  const double m = steps * (L.cw / 16) * 32 / 2100.0;
  if (h->ks == 5) return {1.15 * m, 1.15 * m, h->n_cu};
  if (fp8) return {1.2 * m + 10.0, 2.9 * m + 6.0, 2ll * h->n_cu};
  return {1.55 * m + (L.cw == 64 ? 11.0 : 4.0), 2.55 * m + 16.0, 2ll * h->n_cu};
}

double big_us(const BigTime& b, long long units) {  // units <= b.round
  const double half = b.round / 2.0;
  return units <= half ? b.t1 : b.t1 + (b.t2 - b.t1) * (0.5 + 0.5 * (units - half) / half);
}

// Launches of samples b0 .. b0 + nb - 1 (every per-sample pointer moved on).
pd::HiddenCall layer_call(const pd_predecoder* h, Workspace& ws, const Tiling& t, const LayerRun& L, float* logits,
                          int b0, int nb, hipStream_t st) {
  const Geom& g = h->g;
  const int esz = h->dtype == PD_DTYPE_FP8 ? 1 : 2;  // bytes per activation value
  const long long pv = (long long)b0 * g.S;          // padded voxels before sample b0
  pd::HiddenCall c{};
  c.g = &g;
  c.tl = &t;
  c.cin = L.cin;
  c.cout = L.cout;
  c.act = L.act;
  c.x = (const char*)L.x + pv * L.cin * esz;
  c.y = L.y ? (char*)L.y + pv * L.cout * esz : nullptr;
  c.ystride = L.cout;
  c.wfrag = L.wfrag;
  c.bias = L.bias;
  c.epi = L.epi;
  c.head_w = L.head_w;
  c.head_b = L.head_b;
  c.tables = h->tables;
  c.nib = ws.nib + (long long)b0 * g.V;
  c.logits = logits ? logits + (long long)b0 * 4 * g.T * g.H * g.H : nullptr;
  c.batch = nb;
  c.n_workgroups = h->n_cu * pd::conv_hidden_workgroups_per_cu(h->ks);
  c.sched = ws.sched;
  c.sc = !L.sc ? nullptr : (const uint16_t*)((const char*)L.sc + pv * L.sc_stride * (L.head_w ? 2 : esz));
  c.sc_stride = L.sc_stride;
  c.ks = h->ks;
  c.slice_width = L.cw;
  c.stream = st;
  return c;
}

pd_status run_small(const pd_predecoder* h, Workspace& ws, const LayerRun& L, const pd::SmallPlan& plan, float* logits,
                    int b0, int nb, hipStream_t st) {
  const bool fp8 = h->dtype == PD_DTYPE_FP8;
  Tiling t = h->small[plan.rows / 32 - 2];
  tiling_for_batch(&t, h->g, nb);
  pd::HiddenCall c = layer_call(h, ws, t, L, logits, b0, nb, st);
  const bool head_after = L.epi == 1 && L.cout != 64;
  if (head_after) c.epi = 0;
  pd_status s = check_launch(pd::launch_conv_small(plan, c, fp8));
  if (s == PD_OK && head_after)
    s = check_launch(pd::launch_head(h->g, L.cout, c.y, fp8, L.head_w, L.head_b, h->tables, c.nib, c.logits, nb, st));
  return s;
}

pd_status run_big(const pd_predecoder* h, Workspace& ws, const LayerRun& L, float* logits, int nb, hipStream_t st) {
  Tiling t = h->tiling;
  tiling_for_batch(&t, h->g, nb);
  pd::HiddenCall c = layer_call(h, ws, t, L, logits, 0, nb, st);
  c.cout = L.cw;
  while ((L.cw << c.lsl) < L.cout) ++c.lsl;
  return check_launch(pd::launch_conv_hidden(c, h->dtype == PD_DTYPE_FP8));
}

// The sums of a layer over a batch: samples 0 .. first - 1 in `parts` parts,
// the rest in tail_parts.  When the units fill the persistent kernel's slots
// one to four times over and leave a short remainder, which would take a
// whole unit's time with most of the chip idle, the last few samples take
// parts and run on the small-launch kernel -- for long units only (512 input
// channels): the second launch and the parts cost about 45 us.  (Model 6 at
// 13^3, batch 16: 552 units on 512 slots, the last 2 samples.  Three blocks of
// 512 channels with the remainder apart / in the one launch: bf16 d = 7, batch
// 96 1610 / 1936 us, d = 9, batch 52 1867 / 2005, fp8 d = 7, batch 104 948 / 1056;
// even at worst over 25 sizes.)
constexpr long long kMaxTailRounds = 4;  // past this, a remainder costs little
constexpr double kTailCostUs = 45.0;

struct SumPlan {
  int parts, first, tail_parts;
};

// The tilings of a handle's launches of up to max_batch samples (h->g, h->ks).
void plan_tilings(pd_predecoder* h, int max_batch) {
  h->tiling = plan_tiling(h->g, max_batch, h->ks);
  h->sums = plan_tiling(h->g, max_batch, h->ks, true);
  for (int k = 0; k < 3; ++k) h->small[k] = plan_small(h->g, 64 + 32 * k, h->ks);
}

// Layer l >= 1 of a plain network, but for its buffers: a hidden one, or the
// 5x5x5 output layer.
LayerRun plain_layer(const pd_layer* layers, int n, int l) {
  const pd_layer& a = layers[l];
  LayerRun L{a.c_in, a.c_out, l == n - 1 ? 32 : std::min(a.c_out, 128), a.act};
  L.epi = l == n - 1 ? 2 : 0;
  L.carries_head = l == n - 2 && layers[n - 1].k == 1;
  return L;
}

// conv1 or conv2 (second) of a residual block, but for its buffers.
LayerRun block_conv(const pd_block& B, bool second) {
  const int ci = second ? B.c_mid : B.c_in, co = second ? B.c_out : B.c_mid;
  LayerRun L{ci, co, std::min(co, 128), B.act};
  L.epi = second ? 4 : 0;
  return L;
}

SumPlan sum_plan(const pd_predecoder* h, const LayerRun& L, int batch) {
  const int nsl = L.cout / L.cw;
  auto tiles_of = [&](int nb) {
    Tiling t = h->sums;
    tiling_for_batch(&t, h->g, nb);
    return t.ntiles;
  };
  const long long tiles = tiles_of(batch), units = tiles * nsl;
  const long long round = (long long)h->n_cu * pd::conv_hidden_workgroups_per_cu(h->ks), q = units / round;
  SumPlan p{h->dtype == PD_DTYPE_FP8 ? 1 : conv_parts(h, L, tiles), batch, 1};
  if (p.parts == 1 && q >= 1 && q <= kMaxTailRounds && units % round != 0) {
    // the most first samples whose tiles fit q full rounds (tiles grow with
    // the batch: per sample, or one flat run of batch x V voxels)
    const Tiling& base = h->sums;
    const long long fit = q * round / nsl;  // tiles
    const bool flat = base.mode == 0 && (base.seg_len < 0 || base.tiles_per_seg == 0);
    const long long per = base.mode == 1 ? (long long)base.ntT * base.ntI * base.ntJ : base.tiles_per_seg;
    const long long first = flat ? fit * pd::kTileRows / h->g.V : fit / per;
    if (first >= 1 && first < batch) {
      double unit_us = 0.0;
      const int tail_parts = split_parts(h, tiles_of(batch - (int)first), L.cin, L.cw, nsl, &unit_us);
      if (tail_parts > 1 && unit_us * (1.0 - 1.0 / tail_parts) > kTailCostUs) {
        p.first = (int)first;
        p.tail_parts = tail_parts;
      }
    }
  }
  return p;
}

// A launch of a hidden layer: samples b0 .. b0 + nb - 1, their sums in `parts`
// parts, on the small-launch kernel or the persistent one.
struct Launch {
  int b0, nb, parts;
  bool small;
  pd::SmallPlan plan;
};

// The launches of one hidden layer over a batch: one, or two.
int layer_launches(const pd_predecoder* h, const LayerRun& L, int batch, Launch (&out)[2]) {
  if (L.epi == 2) {  // the 5x5x5 output layer: 4 filters on one block of 32
    out[0] = {0, batch, 4, true, {}};
    (void)small_us(h, L, batch, 4, &out[0].plan);
    return 1;
  }
  const BigTime bt = big_time(h, L);
  auto launch = [&](int b0, int nb, int parts) {
    Launch r{b0, nb, parts, true, {}};
    const double small = small_us(h, L, nb, parts, &r.plan);
    Tiling t = h->tiling;
    tiling_for_batch(&t, h->g, nb);
    const long long units = t.ntiles * (L.cout / L.cw);
    r.small = parts > 1 || b0 > 0 || (units <= bt.round && small * 1.05 < big_us(bt, units));
    return r;
  };
  const SumPlan sp = sum_plan(h, L, batch);
  out[0] = launch(0, sp.first, sp.parts);
  if (sp.first == batch) return 1;
  out[1] = launch(sp.first, batch - sp.first, sp.tail_parts);
  return 2;
}

// One hidden layer over the batch.
pd_status run_hidden(const pd_predecoder* h, Workspace& ws, const LayerRun& L, float* logits, int batch,
                     hipStream_t st) {
  Launch r[2];
  const int n = layer_launches(h, L, batch, r);
  pd_status s = PD_OK;
  for (int k = 0; k < n && s == PD_OK; ++k)
    s = r[k].small ? run_small(h, ws, L, r[k].plan, logits, r[k].b0, r[k].nb, st)
                   : run_big(h, ws, L, logits, r[k].nb, st);
  return s;
}

// Workgroups and whether units come from counters, of a layer's launch on the persistent kernel.
bool big_counts(const pd_predecoder* h, const LayerRun& L, int nb) {
  Tiling t = h->tiling;
  tiling_for_batch(&t, h->g, nb);
  const long long units = t.ntiles * (L.cout / L.cw);
  return pd::conv_hidden_counts(
      units, pd::conv_workgroups(units, (long long)h->n_cu * pd::conv_hidden_workgroups_per_cu(h->ks)));
}

// The path of a residual network (Model 6, Sec. VI, Fig. Model8Representation):
// per block, conv1 (+ folded BatchNorm, activation) x -> hb, the shortcut (x,
// or its 1x1x1 projection into pbuf), conv2 (+ folded BatchNorm) hb -> the
// next x with the shortcut added before the activation; the last block's
// conv2 is the output layer (logits, threshold) with the shortcut added.
// Three activation buffers rotate so that x, hb and the output differ.
// stop >= 0: stop after conv number `stop` of the network (counting, block
// by block, conv1, the projection if the block has one, then conv2; the last
// conv2, the output layer, is not counted) and report its output in *at.
pd_status enqueue_resnet(pd_predecoder* h, Workspace& ws, hipStream_t st, const uint64_t* det, int batch,
                         uint64_t* flips, uint64_t* residual, float* logits, hipEvent_t* ev, int stop, StopAt* at) {
  const Geom& g = h->g;
  const int fp8 = h->dtype == PD_DTYPE_FP8;
  const int ae = fp8 ? 1 : 2;  // bytes per activation value
  int e = 0;
  auto mark = [&]() -> pd_status {
    if (ev && hipEventRecord(ev[e++], st) != hipSuccess) return PD_ERR_DEVICE;
    return PD_OK;
  };
  pd_status s;
  if ((s = mark()) != PD_OK) return s;
  if ((s = check_launch(pd::launch_unpack(g, h->tables, det, batch, ws.planes, 1, 0, st))) != PD_OK) return s;
  const void* x = ws.planes;
  int xi = -1;     // index of x in ws.act (-1: the planes)
  int conv = 0;    // convs run so far (the numbering of `stop`)
  auto stopped = [&](const void* buf, int row_bytes) {
    if (conv++ != stop) return false;
    at->buf = buf;
    at->row_bytes = row_bytes;
    return true;
  };
  const int nb = (int)h->blocks.size();
  for (int k = 0; k < nb; ++k) {
    if ((s = mark()) != PD_OK) return s;
    const pd_block& B = h->blocks[k];
    const bool last = k == nb - 1;
    const int hi = (xi + 1) % 3, yi = (xi + 2 + (xi < 0 ? 1 : 0)) % 3;
    void* hb = ws.act[hi];
    void* yb = ws.act[yi];
    if ((s = prepare_rows(ws, hi, B.c_mid * ae, st)) != PD_OK) return s;
    if (!last && (s = prepare_rows(ws, yi, B.c_out * ae, st)) != PD_OK) return s;
    // conv1: x -> hb (a layer wider than 128 channels: slices of 128 output
    // channels, each with its fragments, biases (fp8: and scales) and output
    // columns; the hidden kernel runs all of them in one launch)
    {
      const int nsl = B.c_mid > 128 ? B.c_mid / 128 : 1, cw = B.c_mid / nsl;
      if (k == 0) {
        // layer 1 (fp8: bf16 matrix work on the dequantised weights, E4M3 output)
        s = check_launch(pd::launch_conv_first(g, B.c_in, cw, nsl, h->wslice[2 * k], B.act, x, nullptr, hb, B.c_mid,
                                               h->wdev[2 * k], h->bdev[2 * k], batch, fp8, 3, st));
      } else {
        LayerRun L = block_conv(B, false);
        L.x = x;
        L.y = hb;
        L.wfrag = h->wdev[2 * k];
        L.bias = h->bdev[2 * k];
        s = run_hidden(h, ws, L, nullptr, batch, st);
      }
      if (s != PD_OK) return s;
      if (stopped(hb, B.c_mid * ae)) return PD_OK;
    }
    // shortcut: the block input, or its 1x1x1 projection -- computed by the
    // epilogue of conv2 from an input of a few channels (the first block)
    // or by the output conv (the last block, its fragments built at create),
    // else by its own kernel (bf16), which also serves a caller that stops
    // at the projection
    const uint16_t* sc = (const uint16_t*)x;
    int sc_stride = B.c_in;
    const float* pw = nullptr;  // set: conv2 projects sc itself
    const float* pb = nullptr;
    if (h->proj_w[k]) {
      const bool fuse = (last ? h->out_proj_frag != nullptr : B.c_in <= 8) && stop != conv;
      if (fuse) {
        pw = h->proj_w[k];
        pb = h->proj_b[k];
        ++conv;  // the projection's stop number
      } else {
        if (fp8) return PD_ERR_UNSUPPORTED;  // no stored fp8 projection
        s = check_launch(pd::launch_proj(g, x, B.c_in, B.c_in, h->proj_w[k], h->proj_b[k], B.c_out, ws.pbuf,
                                         B.c_out, batch, st));
        if (s != PD_OK) return s;
        sc = (const uint16_t*)ws.pbuf;
        sc_stride = B.c_out;
        if (stopped(ws.pbuf, B.c_out * 2)) return PD_OK;
      }
    }
    // conv2: hb -> the next x (or the logits) with the shortcut added
    if (last && pw) {  // the projection fused into the output conv
      s = check_launch(pd::launch_conv_out(g, B.c_mid, hb, h->wdev[2 * k + 1], h->bdev[2 * k + 1], h->tables,
                                           ws.nib, logits, batch, h->n_cu, fp8, nullptr, 0, x, h->out_proj_frag,
                                           h->out_proj_bias, st));
    } else if (last) {
      s = check_launch(pd::launch_conv_out(g, B.c_mid, hb, h->wdev[2 * k + 1], h->bdev[2 * k + 1], h->tables,
                                           ws.nib, logits, batch, h->n_cu, fp8, sc, sc_stride, nullptr, nullptr,
                                           nullptr, st));
    } else {  // slices as for conv1, each also with its shortcut channels (or projection rows)
      LayerRun L = block_conv(B, true);
      L.x = hb;
      L.y = yb;
      L.wfrag = h->wdev[2 * k + 1];
      L.bias = h->bdev[2 * k + 1];
      L.head_w = pw;
      L.head_b = pb;
      L.sc = sc;
      L.sc_stride = sc_stride;
      s = run_hidden(h, ws, L, nullptr, batch, st);
    }
    if (s != PD_OK) return s;
    if (!last && stopped(yb, B.c_out * ae)) return PD_OK;
    x = yb;
    xi = yi;
  }
  if (stop >= 0) return PD_ERR_INVALID_ARG;  // no such conv
  if ((s = mark()) != PD_OK) return s;
  if ((s = check_launch(pd::launch_residual_pack(g, h->tables, det, ws.nib, flips, residual, batch, st))) != PD_OK)
    return s;
  return mark();
}

// Whether layer 1 unpacks the events itself (small launches; not the fp32 one,
// nor a plaquette network's only hidden layer, which carries the head unless
// the run stops at it).
bool layer1_unpacks(const pd_predecoder* h, int batch, int stop) {
  if (!h->blocks.empty() || h->dtype == PD_DTYPE_FP32) return false;
  const bool single = h->layers.size() == 2 && h->layers[1].k == 1 && h->layers[0].c_in == 2 && stop < 0;
  return !single && pd::conv_first_fuses(h->g, batch, h->ks);
}

// Enqueues the whole path in workspace ws.  ev (optional) receives one event
// record before each stage and one after the last.  stop >= 0: stop after
// that hidden layer (residual networks: that conv, see enqueue_resnet), whose
// output activations are then written (no head fused into it) and reported
// in *at.
pd_status enqueue_run(pd_predecoder* h, Workspace& ws, hipStream_t st, const uint64_t* det, int batch,
                      uint64_t* flips, uint64_t* residual, float* logits, hipEvent_t* ev, int stop = -1,
                      StopAt* at = nullptr) {
  if (!h->blocks.empty()) return enqueue_resnet(h, ws, st, det, batch, flips, residual, logits, ev, stop, at);
  const Geom& g = h->g;
  const int fp32 = h->dtype == PD_DTYPE_FP32;
  const int fp8 = h->dtype == PD_DTYPE_FP8;
  const int aelem = fp8 ? 1 : 2;  // bytes per activation value (MFMA paths)
  const int n = (int)h->layers.size();
  // the last layer: a 1x1x1 head (fused into the last hidden layer's
  // epilogue on the MFMA paths) or a 3x3x3 (5x5x5) output layer of its own
  const bool out3 = h->layers[n - 1].k > 1;
  const int ks = h->ks;
  int e = 0;
  auto mark = [&]() -> pd_status {
    if (ev && hipEventRecord(ev[e++], st) != hipSuccess) return PD_ERR_DEVICE;
    return PD_OK;
  };
  pd_status s;
  if ((s = mark()) != PD_OK) return s;
  const bool fused = layer1_unpacks(h, batch, stop);
  if (!fused) s = check_launch(pd::launch_unpack(g, h->tables, det, batch, ws.planes, 1, fp32, st));
  if (s != PD_OK) return s;
  const void* x = ws.planes;
  Tiling tl = h->tiling;
  if (!fp32) tiling_for_batch(&tl, g, batch);
  bool head_done = false;  // nibbles written by a fused head
  for (int l = 0; l < n - 1; ++l) {
    if ((s = mark()) != PD_OK) return s;
    void* y = ws.act[l & 1];
    const pd_layer& L = h->layers[l];
    const int row_bytes = L.c_out * (fp32 ? 4 : aelem);
    if ((s = prepare_rows(ws, l & 1, row_bytes, st)) != PD_OK) return s;
    const bool fuse_head = !out3 && l == n - 2 && stop < 0;  // (a run that stops at the layer does not carry the head)
    if (fp32) {
      s = check_launch(pd::launch_conv_fp32(g, L.c_in, L.c_out, L.act, (const float*)x, (float*)y,
                                            (const float*)h->wdev[l], h->bdev[l], fuse_head ? 1 : 0, h->head_w,
                                            h->head_b, h->tables, ws.nib, logits, batch, h->n_cu, st));
    } else if (l == 0 && fuse_head && L.c_in == 2) {  // one hidden layer: layer 1 carries the head
      s = check_launch(pd::launch_conv_single(g, tl, L.c_out, L.act, x, h->wdev[l], h->bdev[l], h->head_w,
                                              h->head_b, h->tables, ws.nib, logits, batch, h->n_cu, st));
      head_done = true;
    } else {
      // a 256-wide layer runs as two slices of 128 output channels over the
      // same input (slice k: its fragments, biases (fp8: and scales) and
      // output channels)
      const int nsl = h->wslice[l] ? 2 : 1, cw = L.c_out / nsl;
      if (l == 0) {
        const pd::PackedEvents pe{h->tables, det};
        s = check_launch(pd::launch_conv_first(g, L.c_in, cw, nsl, h->wslice[l], L.act, x, fused ? &pe : nullptr, y,
                                               L.c_out, h->wdev[l], h->bdev[l], batch, fp8, ks, st));
      } else {  // the last hidden layer may carry the head and the threshold in its epilogue
        LayerRun R = plain_layer(h->layers.data(), n, l);
        R.x = x;
        R.y = y;
        R.wfrag = h->wdev[l];
        R.bias = h->bdev[l];
        R.epi = fuse_head ? 1 : 0;
        R.head_w = h->head_w;
        R.head_b = h->head_b;
        s = run_hidden(h, ws, R, logits, batch, st);
      }
      head_done = fuse_head && l > 0;
    }
    if (fp32) head_done = fuse_head;
    if (s != PD_OK) return s;
    if (l == stop) {
      at->buf = y;
      at->row_bytes = row_bytes;
      return PD_OK;
    }
    x = y;
  }
  if (stop >= 0) return PD_ERR_INVALID_ARG;  // no such hidden layer
  if ((s = mark()) != PD_OK) return s;
  if (out3 && h->layers[n - 1].k == 3) {
    const pd_layer& L = h->layers[n - 1];
    s = check_launch(pd::launch_conv_out(g, L.c_in, x, h->wdev[n - 1], h->bdev[n - 1], h->tables, ws.nib, logits,
                                         batch, h->n_cu, fp8, nullptr, 0, nullptr, nullptr, nullptr, st));
  } else if (out3) {
    LayerRun R = plain_layer(h->layers.data(), n, n - 1);
    R.x = x;
    R.wfrag = h->wdev[n - 1];
    R.bias = h->bdev[n - 1];
    s = run_hidden(h, ws, R, logits, batch, st);
  } else if (!head_done) {  // a one-hidden-layer network on the paper's layout
    s = check_launch(pd::launch_head(g, h->layers[n - 1].c_in, x, 0, h->head_w, h->head_b, h->tables, ws.nib, logits,
                                     batch, st));
  }
  if (s != PD_OK) return s;
  if ((s = mark()) != PD_OK) return s;
  s = check_launch(pd::launch_residual_pack(g, h->tables, det, ws.nib, flips, residual, batch, st));
  if (s != PD_OK) return s;
  return mark();
}

// Number of convs predecoder_activations can stop after: the hidden layers,
// or for a residual network every conv but the output layer (conv1, the
// projection if any, conv2 per block).
int n_stop_points(const pd_predecoder* h) {
  if (h->blocks.empty()) return (int)h->layers.size() - 1;
  int n = 0;
  for (const pd_block& B : h->blocks) n += 2 + (B.c_in != B.c_out ? 1 : 0);
  return n - 1;
}

}  // namespace

extern "C" {

// For the tests: workgroups of 256 threads of the head's kernel.
int64_t pd_head_blocks(int64_t voxels, int32_t c_in, int32_t fp8) { return pd::head_blocks(voxels, c_in, fp8); }

// For the tests: the launches that a network's layers (blocks given: a
// residual network's convs) after the first take at `batch` samples on a
// handle for max_batch, planned without a device for one of n_cu compute
// units.  out: per launch 6 numbers -- the layer (conv1 and conv2 of block k:
// 2 k and 2 k + 1), its samples, the tile's voxels (256: the persistent
// kernel) and channels, the K parts of its sums, whether units come from
// counters; fp32: a wave's voxels and channels.  Returns the launches, -1 for
// a network that is not supported.
int32_t pd_plan_launches(const pd_layer* layers, int32_t n_layers, const pd_block* blocks, int32_t n_blocks, int32_t d,
                         int32_t T, int32_t dtype, int32_t layout, int32_t batch, int32_t max_batch, int32_t n_cu,
                         int32_t* out, int32_t capacity) {
  pd_predecoder h;
  h.dtype = dtype;
  h.n_cu = n_cu;
  h.ks = blocks ? 3 : network_ks(layers);
  h.g = make_geom(d, T, layout, 0, 0, (h.ks - 1) / 2);
  if (!blocks && !supported(h.g, layers, n_layers, dtype)) return -1;
  if (blocks) h.blocks.assign(blocks, blocks + n_blocks);
  int n = 0;
  auto put = [&](int l, int nb, int rows, int cols, int parts, int counts) {
    if (n < capacity) {
      const int32_t row[6] = {l, nb, rows, cols, parts, counts};
      std::memcpy(out + 6 * n, row, sizeof row);
    }
    ++n;
  };
  if (dtype == PD_DTYPE_FP32) {
    for (int l = 0; l < n_layers - 1; ++l) {
      const pd::Fp32Blocks b =
          pd::conv_fp32_blocks((long long)batch * h.g.V, layers[l].c_out, l == n_layers - 2, n_cu);
      put(l, batch, 16 * b.mb, 16 * b.nb, 1, 0);
    }
    return n;
  }
  plan_tilings(&h, max_batch);
  auto layer = [&](int l, const LayerRun& L) {
    Launch r[2];
    const int k = layer_launches(&h, L, batch, r);
    for (int q = 0; q < k; ++q)
      put(l, r[q].nb, r[q].small ? r[q].plan.rows : pd::kTileRows, r[q].small ? r[q].plan.cols : L.cw, r[q].parts,
          !r[q].small && big_counts(&h, L, r[q].nb));
  };
  if (blocks) {
    for (int k = 0; k < n_blocks; ++k) {
      if (k > 0) layer(2 * k, block_conv(blocks[k], false));
      if (k < n_blocks - 1) layer(2 * k + 1, block_conv(blocks[k], true));
    }
  } else {
    const bool out5 = layers[n_layers - 1].k == 5;
    for (int l = 1; l < n_layers - (out5 ? 0 : 1); ++l) layer(l, plain_layer(layers, n_layers, l));
  }
  return n;
}

const char* predecoder_status_string(pd_status s) {
  switch (s) {
    case PD_OK: return "ok";
    case PD_ERR_INVALID_ARG: return "invalid argument";
    case PD_ERR_UNSUPPORTED: return "unsupported shape";
    case PD_ERR_OUT_OF_MEMORY: return "out of device memory";
    case PD_ERR_DEVICE: return "device error";
    case PD_ERR_TOO_LARGE: return "batch too large for the library's static scratch array";
  }
  return "unknown status";
}

int64_t predecoder_det_words(int32_t d, int32_t T) {
  if (d < 1 || T < 1) return -1;
  return ((int64_t)T * ((int64_t)d * d - 1) + 63) / 64;
}

int64_t predecoder_flip_words(int32_t d, int32_t T) {
  if (d < 1 || T < 1) return -1;
  return ((int64_t)T * (3 * (int64_t)d * d - 1) + 63) / 64;
}

size_t predecoder_weight_count(const pd_layer* layers, int32_t n_layers) {
  if (!layers || n_layers < 1) return 0;
  size_t n = 0;
  for (int i = 0; i < n_layers; ++i) {
    const pd_layer& l = layers[i];
    if (l.c_in < 1 || l.c_out < 1 || l.k < 1) return 0;
    n += (size_t)l.c_out * l.c_in * l.k * l.k * l.k + l.c_out;
  }
  return n;
}

int32_t predecoder_num_stages(const pd_predecoder* h) {
  if (!h) return -1;
  return (int32_t)(h->blocks.empty() ? h->layers.size() : h->blocks.size()) + 2;
}

pd_status predecoder_create(const float* weights, size_t n_weights, int32_t d, int32_t T,
                            const pd_layer* layers, int32_t n_layers, int32_t dtype, int32_t max_batch,
                            pd_predecoder** out) {
  return predecoder_create_ex(weights, n_weights, d, T, layers, n_layers, dtype, max_batch, nullptr, out);
}

pd_status predecoder_create_ex(const float* weights, size_t n_weights, int32_t d, int32_t T,
                               const pd_layer* layers, int32_t n_layers, int32_t dtype, int32_t max_batch,
                               const pd_options* opts, pd_predecoder** out) {
  if (!out) return PD_ERR_INVALID_ARG;
  *out = nullptr;
  if (!weights || !layers) return PD_ERR_INVALID_ARG;
  if (d < 3 || (d % 2) == 0 || T < 1) return PD_ERR_INVALID_ARG;
  if (dtype != PD_DTYPE_FP32 && dtype != PD_DTYPE_BF16 && dtype != PD_DTYPE_FP8) return PD_ERR_INVALID_ARG;
  if (max_batch < 1) return PD_ERR_INVALID_ARG;
  const pd_options o = opts ? *opts : pd_options{PD_LAYOUT_PLAQUETTE, PD_BOUNDARY_NONE, PD_BOUNDARY_NONE};
  if (o.layout != PD_LAYOUT_PLAQUETTE && o.layout != PD_LAYOUT_PAPER) return PD_ERR_INVALID_ARG;
  if (o.first_round < PD_BOUNDARY_NONE || o.first_round > PD_BOUNDARY_X || o.last_round < PD_BOUNDARY_NONE ||
      o.last_round > PD_BOUNDARY_X)
    return PD_ERR_INVALID_ARG;
  // the plaquette layout has no geometric channels to clear
  if (o.layout == PD_LAYOUT_PLAQUETTE && (o.first_round != PD_BOUNDARY_NONE || o.last_round != PD_BOUNDARY_NONE))
    return PD_ERR_INVALID_ARG;
  if (!layer_chain_ok(layers, n_layers, o.layout)) return PD_ERR_INVALID_ARG;
  if (n_weights != predecoder_weight_count(layers, n_layers)) return PD_ERR_INVALID_ARG;
  const int ks = network_ks(layers);
  // the zero halo holds every tap of a layer: one voxel, two for 5x5x5 layers
  Geom g = make_geom(d, T, o.layout, o.first_round, o.last_round, (ks - 1) / 2);
  if (!supported(g, layers, n_layers, dtype)) return PD_ERR_UNSUPPORTED;
  // kernels index voxels of a batch with 32-bit integers
  if ((long long)max_batch * g.V >= (1ll << 31) || (long long)max_batch * (g.Wd + g.Wf) >= (1ll << 31) ||
      (long long)max_batch * g.S >= (1ll << 31) ||
      (long long)max_batch * (T + 2) * pd::line_plane(g) >= (1ll << 31))
    return PD_ERR_UNSUPPORTED;

  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || ndev < 1) {
    (void)hipGetLastError();
    return PD_ERR_DEVICE;
  }
  pd_predecoder* h = new (std::nothrow) pd_predecoder();
  if (!h) return PD_ERR_OUT_OF_MEMORY;
  h->g = g;
  h->dtype = dtype;
  h->max_batch = max_batch;
  h->layers.assign(layers, layers + n_layers);
  h->ks = ks;
  if (hipGetDevice(&h->device) != hipSuccess ||
      hipDeviceGetAttribute(&h->n_cu, hipDeviceAttributeMultiprocessorCount, h->device) != hipSuccess ||
      h->n_cu < 1) {
    (void)hipGetLastError();
    delete h;
    return PD_ERR_DEVICE;
  }
  int cmax = 2;
  for (int i = 0; i < n_layers - 1; ++i) cmax = std::max(cmax, (int)layers[i].c_out);
  h->cmax = cmax;
  if (dtype != PD_DTYPE_FP32) {
    plan_tilings(h, max_batch);
    const int max_span = ks == 3 ? std::min(pd::conv_single_max_span(), pd::conv_hidden_max_span(3))
                                 : pd::conv_hidden_max_span(5);
    if (h->tiling.span <= 0 || h->tiling.span > max_span) {
      delete h;
      return PD_ERR_UNSUPPORTED;
    }
  }

  pd_status s = PD_OK;
  // planes: fp32 or bf16; activations: fp32, bf16 or E4M3
  const size_t elem = dtype == PD_DTYPE_FP32 ? 4 : 2;
  const size_t aelem = dtype == PD_DTYPE_FP32 ? 4 : (dtype == PD_DTYPE_FP8 ? 1 : 2);
  const size_t vox = (size_t)max_batch * (size_t)g.S;
  auto fail = [&](pd_status st) {
    free_all(h);
    delete h;
    return st;
  };
  const size_t cin0 = (size_t)layers[0].c_in;
  if ((s = dev_alloc(&h->ws.planes, vox * cin0 * elem)) != PD_OK) return fail(s);
  h->ws.act_bytes = vox * cmax * aelem;
  if ((s = dev_alloc(&h->ws.act[0], vox * cmax * aelem)) != PD_OK) return fail(s);
  if ((s = dev_alloc(&h->ws.act[1], vox * cmax * aelem)) != PD_OK) return fail(s);
  if ((s = dev_alloc(&h->ws.nib, (size_t)max_batch * g.V)) != PD_OK) return fail(s);
  if (dtype != PD_DTYPE_FP32) {
    if ((s = dev_alloc(&h->ws.sched, kSchedWords * 4)) != PD_OK) return fail(s);
    if (hipMemset(h->ws.sched, 0, kSchedWords * 4) != hipSuccess) return fail(PD_ERR_DEVICE);
  }
  std::vector<int32_t> tab = build_tables(g);
  if ((s = upload(&h->tables, tab.data(), tab.size() * sizeof(int32_t))) != PD_OK) return fail(s);
  if (hipMemset(h->ws.planes, 0, vox * cin0 * elem) != hipSuccess ||
      hipMemset(h->ws.act[0], 0, vox * cmax * aelem) != hipSuccess ||
      hipMemset(h->ws.act[1], 0, vox * cmax * aelem) != hipSuccess)
    return fail(PD_ERR_DEVICE);

  const float* src = weights;
  for (int i = 0; i < n_layers; ++i) {
    const pd_layer& L = layers[i];
    const size_t nw = (size_t)L.c_out * L.c_in * L.k * L.k * L.k;
    const float* w = src;
    const float* b = src + nw;
    src += nw + L.c_out;
    // fp8: weight codes, per-channel scales and the values they stand for
    std::vector<uint8_t> codes;
    std::vector<float> scale, wq;
    if (dtype == PD_DTYPE_FP8) quantize_e4m3(w, L.c_out, nw / L.c_out, &codes, &scale, &wq);
    if (i == n_layers - 1 && L.k == 3) {  // a 3x3x3 output layer: rows (tap, filter)
      if (!pd::conv_out_supported(L.c_in, dtype == PD_DTYPE_FP8, 3, g.H)) return fail(PD_ERR_UNSUPPORTED);
      std::vector<uint8_t> f = out_fragments(w, codes.data(), L.c_in, dtype == PD_DTYPE_FP8);
      void* wd = nullptr;
      s = upload(&wd, f.data(), f.size());
      h->wdev.push_back(wd);
      h->wslice.push_back(0);
      if (s != PD_OK) return fail(s);
      std::vector<float> bp(8, 1.0f);
      for (int o2 = 0; o2 < 4; ++o2) {
        bp[o2] = b[o2];
        if (dtype == PD_DTYPE_FP8) bp[4 + o2] = scale[o2];
      }
      float* bd = nullptr;
      s = upload(&bd, bp.data(), bp.size() * 4);
      h->bdev.push_back(bd);
      if (s != PD_OK) return fail(s);
      break;
    }
    if (i == n_layers - 1 && L.k > 1) {  // a 5x5x5 output layer: 4 filters padded to one block of 32
      void* wd = nullptr;
      if (dtype == PD_DTYPE_FP8) {
        std::vector<uint8_t> f = conv_fragments_fp8(codes.data(), L.c_in, L.c_out);
        s = upload(&wd, f.data(), f.size());
      } else {
        std::vector<uint16_t> f = conv_fragments(w, L.c_in, L.c_out, L.k);
        s = upload(&wd, f.data(), f.size() * 2);
      }
      h->wdev.push_back(wd);
      h->wslice.push_back(0);
      if (s != PD_OK) return fail(s);
      // biases of the 32 padded channels, then (fp8) their weight scales
      std::vector<float> bp(64, 0.0f);
      for (int o2 = 0; o2 < L.c_out; ++o2) {
        bp[o2] = b[o2];
        bp[32 + o2] = dtype == PD_DTYPE_FP8 ? scale[o2] : 1.0f;
      }
      float* bd = nullptr;
      s = upload(&bd, bp.data(), bp.size() * 4);
      h->bdev.push_back(bd);
      if (s != PD_OK) return fail(s);
      break;
    }
    if (i == n_layers - 1) {
      std::vector<float> hw((size_t)4 * L.c_in);
      for (int o = 0; o < 4; ++o)
        for (int c = 0; c < L.c_in; ++c) {
          float v = w[(size_t)o * L.c_in + c];
          hw[(size_t)o * L.c_in + c] =
              dtype == PD_DTYPE_BF16 ? bf16_value(v) : (dtype == PD_DTYPE_FP8 ? wq[(size_t)o * L.c_in + c] : v);
        }
      if ((s = upload(&h->head_w, hw.data(), hw.size() * 4)) != PD_OK) return fail(s);
      if ((s = upload(&h->head_b, b, 4 * sizeof(float))) != PD_OK) return fail(s);
      break;
    }
    void* wd = nullptr;
    size_t slice = 0;
    std::vector<float> bias_dev(b, b + L.c_out);
    if (dtype == PD_DTYPE_FP8 && i > 0) {
      // E4M3 fragments; per 128-channel slice: its biases, then its scales
      const int cw = L.c_out == 256 ? 128 : L.c_out;
      std::vector<uint8_t> f = conv_fragments_fp8(codes.data(), L.c_in, cw);
      bias_dev.assign(b, b + cw);
      bias_dev.insert(bias_dev.end(), scale.begin(), scale.begin() + cw);
      if (L.c_out == 256) {
        slice = f.size();
        std::vector<uint8_t> f2 = conv_fragments_fp8(codes.data() + (size_t)128 * L.c_in * 27, L.c_in, 128);
        f.insert(f.end(), f2.begin(), f2.end());
        bias_dev.insert(bias_dev.end(), b + 128, b + 256);
        bias_dev.insert(bias_dev.end(), scale.begin() + 128, scale.end());
      }
      s = upload(&wd, f.data(), f.size());
    } else if (dtype != PD_DTYPE_FP32) {
      // bf16 fragments (fp8 layer 1: of the E4M3 values times their scales,
      // exact in bf16)
      const float* wv = dtype == PD_DTYPE_FP8 ? wq.data() : w;
      std::vector<uint16_t> f;
      if (L.c_out == 256) {  // two slices of 128 output channels, back to back
        f = conv_fragments(wv, L.c_in, 128);
        slice = f.size() * 2;
        std::vector<uint16_t> f2 = conv_fragments(wv + (size_t)128 * L.c_in * 27, L.c_in, 128);
        f.insert(f.end(), f2.begin(), f2.end());
      } else {
        f = conv_fragments(wv, L.c_in, L.c_out, L.k);
      }
      s = upload(&wd, f.data(), f.size() * 2);
    } else {
      const int head = i == n_layers - 2;
      std::vector<float> r = pd::conv_fp32_fragments(w, L.c_in, L.c_out, head);
      bias_dev = pd::conv_fp32_bias(b, L.c_out, head);
      s = upload(&wd, r.data(), r.size() * 4);
    }
    h->wdev.push_back(wd);
    h->wslice.push_back(slice);
    if (s != PD_OK) return fail(s);
    float* bd = nullptr;
    s = upload(&bd, bias_dev.data(), bias_dev.size() * 4);
    h->bdev.push_back(bd);
    if (s != PD_OK) return fail(s);
  }
  if (hipDeviceSynchronize() != hipSuccess) return fail(PD_ERR_DEVICE);
  *out = h;
  return PD_OK;
}

size_t predecoder_resnet_weight_count(const pd_block* b, int32_t n) {
  if (!b || n < 1) return 0;
  size_t total = 0;
  for (int k = 0; k < n; ++k) {
    const size_t ci = b[k].c_in, cm = b[k].c_mid, co = b[k].c_out;
    if (b[k].c_in < 1 || b[k].c_mid < 1 || b[k].c_out < 1) return 0;
    total += cm * ci * 27 + cm + 4 * cm + co * cm * 27 + co + 4 * co;
    if (ci != co) total += co * ci + co;
  }
  return total;
}

pd_status predecoder_create_resnet(const float* weights, size_t n_weights, int32_t d, int32_t T,
                                   const pd_block* blocks, int32_t n_blocks, int32_t dtype, int32_t max_batch,
                                   const pd_options* opts, pd_predecoder** out) {
  if (!out) return PD_ERR_INVALID_ARG;
  *out = nullptr;
  if (!weights || !blocks || n_blocks < 1) return PD_ERR_INVALID_ARG;
  if (d < 3 || (d % 2) == 0 || T < 1 || max_batch < 1) return PD_ERR_INVALID_ARG;
  if (dtype != PD_DTYPE_FP32 && dtype != PD_DTYPE_BF16 && dtype != PD_DTYPE_FP8) return PD_ERR_INVALID_ARG;
  const pd_options o = opts ? *opts : pd_options{PD_LAYOUT_PLAQUETTE, PD_BOUNDARY_NONE, PD_BOUNDARY_NONE};
  if (o.layout != PD_LAYOUT_PLAQUETTE && o.layout != PD_LAYOUT_PAPER) return PD_ERR_INVALID_ARG;
  if (o.first_round < PD_BOUNDARY_NONE || o.first_round > PD_BOUNDARY_X || o.last_round < PD_BOUNDARY_NONE ||
      o.last_round > PD_BOUNDARY_X)
    return PD_ERR_INVALID_ARG;
  if (o.layout == PD_LAYOUT_PLAQUETTE && (o.first_round != PD_BOUNDARY_NONE || o.last_round != PD_BOUNDARY_NONE))
    return PD_ERR_INVALID_ARG;
  // the chain: input channels of the layout, widths that meet, 4 outputs
  if (blocks[0].c_in != (o.layout == PD_LAYOUT_PAPER ? 4 : 2) || blocks[n_blocks - 1].c_out != 4)
    return PD_ERR_INVALID_ARG;
  for (int k = 0; k < n_blocks; ++k) {
    const pd_block& B = blocks[k];
    if (B.c_in < 1 || B.c_mid < 1 || B.c_out < 1 || B.act < 0 || B.act > 2) return PD_ERR_INVALID_ARG;
    if (k > 0 && B.c_in != blocks[k - 1].c_out) return PD_ERR_INVALID_ARG;
  }
  if (n_weights != predecoder_resnet_weight_count(blocks, n_blocks)) return PD_ERR_INVALID_ARG;
  // what the kernels run: bf16 or fp8; widths 64, 128, 256 or 512 with
  // c_out = c_mid inside the network; fp8: projections only where they are
  // fused (the first block, from its few input channels, and the last, with
  // c_in = c_mid)
  if (dtype != PD_DTYPE_BF16 && dtype != PD_DTYPE_FP8) return PD_ERR_UNSUPPORTED;
  if (dtype == PD_DTYPE_FP8)
    for (int k = 0; k < n_blocks; ++k) {
      const pd_block& B = blocks[k];
      if (B.c_in == B.c_out) continue;
      const bool first_ok = k == 0 && B.c_in <= 8 && n_blocks > 1;
      const bool last_ok = k == n_blocks - 1 && B.c_in == B.c_mid;
      if (!first_ok && !last_ok) return PD_ERR_UNSUPPORTED;
    }
  auto width_ok = [](int c) { return c == 64 || c == 128 || c == 256 || c == 512; };
  // conv1 of a later block runs the hidden kernel from c_in to slices of
  // min(c_mid, 128) channels: the instantiated pairs
  auto conv1_ok = [](int ci, int cw) {
    return (ci == 64 && (cw == 64 || cw == 128)) || (ci == 128 && (cw == 64 || cw == 128)) ||
           (ci == 256 && (cw == 64 || cw == 128)) || (ci == 512 && cw == 128);
  };
  for (int k = 0; k < n_blocks; ++k) {
    const pd_block& B = blocks[k];
    if (!width_ok(B.c_mid)) return PD_ERR_UNSUPPORTED;
    if (k < n_blocks - 1 && B.c_out != B.c_mid) return PD_ERR_UNSUPPORTED;
    if (k > 0 && !conv1_ok(B.c_in, B.c_mid > 128 ? 128 : B.c_mid)) return PD_ERR_UNSUPPORTED;
  }
  Geom g = make_geom(d, T, o.layout, o.first_round, o.last_round);
  if (g.d > kMaxD || g.T > kMaxT) return PD_ERR_UNSUPPORTED;
  if ((long long)max_batch * g.V >= (1ll << 31) || (long long)max_batch * (g.Wd + g.Wf) >= (1ll << 31) ||
      (long long)max_batch * g.S >= (1ll << 31) ||
      (long long)max_batch * (T + 2) * pd::line_plane(g) >= (1ll << 31))
    return PD_ERR_UNSUPPORTED;
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || ndev < 1) {
    (void)hipGetLastError();
    return PD_ERR_DEVICE;
  }
  pd_predecoder* h = new (std::nothrow) pd_predecoder();
  if (!h) return PD_ERR_OUT_OF_MEMORY;
  h->g = g;
  h->dtype = dtype;
  h->max_batch = max_batch;
  h->blocks.assign(blocks, blocks + n_blocks);
  if (hipGetDevice(&h->device) != hipSuccess ||
      hipDeviceGetAttribute(&h->n_cu, hipDeviceAttributeMultiprocessorCount, h->device) != hipSuccess ||
      h->n_cu < 1) {
    (void)hipGetLastError();
    delete h;
    return PD_ERR_DEVICE;
  }
  plan_tilings(h, max_batch);
  if (h->tiling.span <= 0 || h->tiling.span > pd::conv_hidden_max_span(3)) {
    delete h;
    return PD_ERR_UNSUPPORTED;
  }
  int cmax = 4, pmax = 4;
  for (int k = 0; k < n_blocks; ++k) {
    cmax = std::max(cmax, std::max((int)blocks[k].c_mid, (int)blocks[k].c_out));
    if (blocks[k].c_in != blocks[k].c_out) pmax = std::max(pmax, (int)blocks[k].c_out);
  }
  h->cmax = cmax;
  h->pmax = pmax;
  pd_status s = PD_OK;
  auto fail = [&](pd_status st) {
    free_all(h);
    delete h;
    return st;
  };
  const size_t vox = (size_t)max_batch * (size_t)g.S;
  const size_t cin0 = (size_t)blocks[0].c_in;
  if ((s = dev_alloc(&h->ws.planes, vox * cin0 * 2)) != PD_OK) return fail(s);
  h->ws.act_bytes = vox * cmax * 2;
  if ((s = dev_alloc(&h->ws.act[0], vox * cmax * 2)) != PD_OK) return fail(s);
  if ((s = dev_alloc(&h->ws.act[1], vox * cmax * 2)) != PD_OK) return fail(s);
  if ((s = dev_alloc(&h->ws.act[2], vox * cmax * 2)) != PD_OK) return fail(s);
  if ((s = dev_alloc(&h->ws.pbuf, vox * pmax * 2)) != PD_OK) return fail(s);
  if ((s = dev_alloc(&h->ws.nib, (size_t)max_batch * g.V)) != PD_OK) return fail(s);
  if ((s = dev_alloc(&h->ws.sched, kSchedWords * 4)) != PD_OK) return fail(s);
  if (hipMemset(h->ws.sched, 0, kSchedWords * 4) != hipSuccess) return fail(PD_ERR_DEVICE);
  std::vector<int32_t> tab = build_tables(g);
  if ((s = upload(&h->tables, tab.data(), tab.size() * sizeof(int32_t))) != PD_OK) return fail(s);
  if (hipMemset(h->ws.planes, 0, vox * cin0 * 2) != hipSuccess || hipMemset(h->ws.act[0], 0, vox * cmax * 2) != hipSuccess ||
      hipMemset(h->ws.act[1], 0, vox * cmax * 2) != hipSuccess || hipMemset(h->ws.act[2], 0, vox * cmax * 2) != hipSuccess ||
      hipMemset(h->ws.pbuf, 0, vox * pmax * 2) != hipSuccess)
    return fail(PD_ERR_DEVICE);
  // weights: per conv, BatchNorm folded in (g = scale / sqrt(var + 1e-5) in
  // fp64; weights fp32(w g), rounded to bf16 by the fragment builder or, on
  // the fp8 path, quantised per output channel to E4M3; bias fp32((b - mean)
  // g + shift))
  const bool fp8 = dtype == PD_DTYPE_FP8;
  const float* src = weights;
  for (int k = 0; k < n_blocks; ++k) {
    const pd_block& B = blocks[k];
    for (int c = 0; c < 2; ++c) {
      const int cin = c == 0 ? B.c_in : B.c_mid, cout = c == 0 ? B.c_mid : B.c_out;
      const size_t nw = (size_t)cout * cin * 27;
      const float* w = src;
      const float* b = src + nw;
      const float* bn = b + cout;  // scale, shift, mean, var
      src += nw + cout + 4 * (size_t)cout;
      std::vector<float> wf(nw), bf(cout > 4 ? cout : 32, 0.0f);
      for (int o2 = 0; o2 < cout; ++o2) {
        const double gg = (double)bn[o2] / std::sqrt((double)bn[3 * cout + o2] + 1e-5);
        for (size_t e = 0; e < (size_t)cin * 27; ++e) wf[o2 * (size_t)cin * 27 + e] = (float)((double)w[o2 * (size_t)cin * 27 + e] * gg);
        bf[o2] = (float)(((double)b[o2] - bn[2 * cout + o2]) * gg + bn[cout + o2]);
      }
      // fp8: the folded weights' E4M3 codes and per-channel scales (and the
      // values they stand for, for layer 1's bf16 fragments)
      std::vector<uint8_t> codes;
      std::vector<float> scale, wq;
      if (fp8) quantize_e4m3(wf.data(), cout, (size_t)cin * 27, &codes, &scale, &wq);
      size_t slice = 0;
      void* wd = nullptr;
      if (c == 1 && k == n_blocks - 1) {  // the output conv, 4 filters: rows (tap, filter)
        if (!pd::conv_out_supported(cin, fp8, 3, g.H)) return fail(PD_ERR_UNSUPPORTED);
        std::vector<uint8_t> f = out_fragments(wf.data(), codes.data(), cin, fp8);
        s = upload(&wd, f.data(), f.size());
        bf.resize(8);
        for (int o2 = 0; o2 < 4; ++o2) bf[4 + o2] = fp8 ? scale[o2] : 1.0f;  // [4] biases, then [4] weight scales
      } else if (fp8 && !(c == 0 && k == 0)) {
        // E4M3 fragments per 128-channel slice; per slice its biases, then its scales
        const int cw = cout > 128 ? 128 : cout, nsl = cout / cw;
        std::vector<uint8_t> f;
        std::vector<float> bd;
        for (int q = 0; q < nsl; ++q) {
          std::vector<uint8_t> fq = conv_fragments_fp8(codes.data() + (size_t)q * cw * cin * 27, cin, cw);
          if (nsl > 1) slice = fq.size();
          f.insert(f.end(), fq.begin(), fq.end());
          bd.insert(bd.end(), bf.begin() + (size_t)q * cw, bf.begin() + (size_t)(q + 1) * cw);
          bd.insert(bd.end(), scale.begin() + (size_t)q * cw, scale.begin() + (size_t)(q + 1) * cw);
        }
        bf = bd;
        s = upload(&wd, f.data(), f.size());
      } else {
        // bf16 fragments (fp8 layer 1: of the E4M3 values times their scales, exact in bf16)
        std::vector<uint16_t> f = fragments_sliced(fp8 ? wq.data() : wf.data(), cin, cout, &slice);
        s = upload(&wd, f.data(), f.size() * 2);
      }
      h->wdev.push_back(wd);
      h->wslice.push_back(slice);
      if (s != PD_OK) return fail(s);
      float* bd = nullptr;
      s = upload(&bd, bf.data(), bf.size() * 4);
      h->bdev.push_back(bd);
      if (s != PD_OK) return fail(s);
    }
    float* pw = nullptr;
    float* pb = nullptr;
    if (B.c_in != B.c_out) {
      // weights: bf16 values, or (fp8) E4M3 codes with per-channel scales and
      // the values they stand for
      const size_t np = (size_t)B.c_out * B.c_in;
      std::vector<uint8_t> pcodes;
      std::vector<float> pscale, pvals;
      if (fp8) {
        quantize_e4m3(src, B.c_out, B.c_in, &pcodes, &pscale, &pvals);
      } else {
        pvals.resize(np);
        for (size_t e = 0; e < np; ++e) pvals[e] = bf16_value(src[e]);
      }
      s = upload(&pw, pvals.data(), np * 4);
      if (s == PD_OK) s = upload(&pb, src + np, (size_t)B.c_out * 4);
      // the last block's projection (c_in = c_mid) runs inside the output
      // conv: fragments [k-step][lane], lane l's row l % 32 (filters 0..3,
      // the rest zero), bf16: ci = 16 k-step + 8 (l / 32) + e; fp8 codes:
      // ci = 64 k-step + 32 (l / 32) + e; then [4] biases and [4] scales
      if (s == PD_OK && k == n_blocks - 1 && B.c_in == B.c_mid) {
        const int kstep = fp8 ? 64 : 16, lb = fp8 ? 32 : 16, per = fp8 ? 32 : 8;
        std::vector<uint8_t> pf(pd::conv_out_proj_fragment_bytes(B.c_in, fp8), 0);
        for (int st = 0; st < B.c_in / kstep; ++st)
          for (int l = 0; l < 64; ++l)
            for (int e = 0; e < per; ++e) {
              const int co = l % 32, ci = st * kstep + per * (l / 32) + e;
              if (co >= B.c_out) continue;
              uint8_t* dst = &pf[((size_t)st * 64 + l) * lb];
              if (fp8) {
                dst[e] = pcodes[(size_t)co * B.c_in + ci];
              } else {
                const uint16_t v = bf16_bits(src[(size_t)co * B.c_in + ci]);
                std::memcpy(dst + 2 * e, &v, 2);
              }
            }
        s = upload(&h->out_proj_frag, pf.data(), pf.size());
        std::vector<float> pbias(8, 1.0f);
        for (int o2 = 0; o2 < 4; ++o2) {
          pbias[o2] = src[np + o2];
          if (fp8) pbias[4 + o2] = pscale[o2];
        }
        if (s == PD_OK) s = upload(&h->out_proj_bias, pbias.data(), pbias.size() * 4);
      }
      src += np + B.c_out;
    }
    h->proj_w.push_back(pw);
    h->proj_b.push_back(pb);
    if (s != PD_OK) return fail(s);
  }
  if (hipDeviceSynchronize() != hipSuccess) return fail(PD_ERR_DEVICE);
  *out = h;
  return PD_OK;
}

pd_status predecoder_run(pd_predecoder* h, void* hip_stream, const uint64_t* det, int32_t batch,
                         uint64_t* flips, uint64_t* residual, float* logits) {
  if (!h || !det || !flips || !residual) return PD_ERR_INVALID_ARG;
  if (batch < 1 || batch > h->max_batch) return PD_ERR_INVALID_ARG;
  return enqueue_run(h, h->ws, (hipStream_t)hip_stream, det, batch, flips, residual, logits, nullptr);
}

}  // extern "C"

namespace pd {

pd_status run_in_region(pd_predecoder* h, hipStream_t st, const uint64_t* det, int batch, uint64_t* flips,
                        uint64_t* residual, float* logits, void* base, size_t bytes) {
  if (!h || !det || !flips || !residual || !base) return PD_ERR_INVALID_ARG;
  if (batch < 1 || batch > h->max_batch) return PD_ERR_INVALID_ARG;
  const Geom& g = h->g;
  const bool resnet = !h->blocks.empty();
  const int fp32 = h->dtype == PD_DTYPE_FP32, fp8 = h->dtype == PD_DTYPE_FP8;
  const size_t elem = fp32 ? 4 : 2;                 // input planes
  const size_t aelem = fp32 ? 4 : (fp8 ? 1 : 2);   // activations
  const size_t cin0 = resnet ? (size_t)h->blocks[0].c_in : (size_t)h->layers[0].c_in;
  const size_t vox = (size_t)batch * (size_t)g.S;
  // regions of 256-byte aligned offsets: planes, activations, projection
  // outputs (residual networks), flip nibbles
  size_t off = 0;
  auto carve = [&](size_t n) {
    const size_t at = (off + 255) & ~(size_t)255;
    off = at + ((n + 255) & ~(size_t)255);
    return at;
  };
  const size_t planes_bytes = vox * cin0 * elem, act_bytes = vox * (size_t)h->cmax * aelem;
  const size_t o_planes = carve(planes_bytes);
  size_t o_act[3] = {carve(act_bytes), carve(act_bytes), 0};
  size_t o_pbuf = 0;
  if (resnet) {
    o_act[2] = carve(act_bytes);
    o_pbuf = carve(vox * (size_t)h->pmax * 2);
  }
  const size_t o_nib = carve((size_t)batch * g.V);
  const size_t o_sched = fp32 ? 0 : carve(kSchedWords * 4);
  if (off > bytes) return PD_ERR_TOO_LARGE;
  char* b = (char*)base;
  Workspace ws;
  ws.planes = b + o_planes;
  for (int k = 0; k < (resnet ? 3 : 2); ++k) ws.act[k] = b + o_act[k];
  ws.pbuf = resnet ? (void*)(b + o_pbuf) : nullptr;
  ws.nib = (uint8_t*)(b + o_nib);
  ws.act_bytes = act_bytes;
  // the zero halos the 3x3x3 layers read: the planes and every activation
  // buffer start all zero (a fill kernel, so that the call can be captured
  // into a graph); the other regions are written before they are read
  pd_status s = check_launch(launch_zero(ws.planes, (planes_bytes + 15) & ~(size_t)15, st));
  for (int k = 0; k < (resnet ? 3 : 2) && s == PD_OK; ++k)
    s = check_launch(launch_zero(ws.act[k], (act_bytes + 15) & ~(size_t)15, st));
  if (!fp32 && s == PD_OK) {  // the hidden kernel's unit counters start at zero (and stay so between launches)
    ws.sched = (uint32_t*)(b + o_sched);
    s = check_launch(launch_zero(ws.sched, kSchedWords * 4, st));
  }
  if (s != PD_OK) return s;
  return enqueue_run(h, ws, st, det, batch, flips, residual, logits, nullptr);
}

}  // namespace pd

extern "C" {

pd_status predecoder_residual(pd_predecoder* h, void* hip_stream, const uint64_t* det,
                              const uint64_t* flips, int32_t batch, uint64_t* residual) {
  if (!h || !det || !flips || !residual) return PD_ERR_INVALID_ARG;
  if (batch < 1 || batch > h->max_batch) return PD_ERR_INVALID_ARG;
  return check_launch(
      pd::launch_residual_from_flips(h->g, h->tables, det, flips, residual, batch, (hipStream_t)hip_stream));
}

pd_status predecoder_activations(pd_predecoder* h, void* hip_stream, const uint64_t* det, int32_t batch,
                                 int32_t layer, void* out) {
  if (!h || !det || !out) return PD_ERR_INVALID_ARG;
  if (batch < 1 || batch > h->max_batch) return PD_ERR_INVALID_ARG;
  if (layer < 0 || layer >= n_stop_points(h)) return PD_ERR_INVALID_ARG;
  if (h->dtype == PD_DTYPE_FP32) return PD_ERR_UNSUPPORTED;
  const hipStream_t st = (hipStream_t)hip_stream;
  StopAt at;
  pd_status s = enqueue_run(h, h->ws, st, det, batch, nullptr, nullptr, nullptr, nullptr, layer, &at);
  if (s != PD_OK) return s;
  return check_launch(pd::launch_extract(h->g, at.buf, at.row_bytes, batch, out, st));
}

pd_status predecoder_unpack(pd_predecoder* h, void* hip_stream, const uint64_t* det, int32_t batch,
                            void* planes) {
  if (!h || !det || !planes) return PD_ERR_INVALID_ARG;
  if (batch < 1 || batch > h->max_batch) return PD_ERR_INVALID_ARG;
  return check_launch(pd::launch_unpack(h->g, h->tables, det, batch, planes, 0,
                                        h->dtype == PD_DTYPE_FP32, (hipStream_t)hip_stream));
}

pd_status predecoder_stage_times(pd_predecoder* h, void* hip_stream, const uint64_t* det, int32_t batch,
                                 uint64_t* flips, uint64_t* residual, int32_t n_iter, float* ms_per_stage) {
  if (!h || !det || !flips || !residual || !ms_per_stage) return PD_ERR_INVALID_ARG;
  if (batch < 1 || batch > h->max_batch || n_iter < 1 || n_iter > 100000) return PD_ERR_INVALID_ARG;
  const int ns = predecoder_num_stages(h);
  const int ne = ns + 1;
  std::vector<hipEvent_t> ev((size_t)n_iter * ne, nullptr);
  pd_status s = PD_OK;
  for (auto& e : ev)
    if (hipEventCreate(&e) != hipSuccess) {
      s = PD_ERR_DEVICE;
      break;
    }
  hipStream_t st = (hipStream_t)hip_stream;
  for (int it = 0; it < n_iter && s == PD_OK; ++it)
    s = enqueue_run(h, h->ws, st, det, batch, flips, residual, nullptr, ev.data() + (size_t)it * ne);
  if (s == PD_OK && hipStreamSynchronize(st) != hipSuccess) s = PD_ERR_DEVICE;
  if (s == PD_OK) {
    for (int k = 0; k < ns; ++k) ms_per_stage[k] = 0.0f;
    for (int it = 0; it < n_iter && s == PD_OK; ++it)
      for (int k = 0; k < ns; ++k) {
        float ms = 0.0f;
        if (hipEventElapsedTime(&ms, ev[(size_t)it * ne + k], ev[(size_t)it * ne + k + 1]) != hipSuccess) {
          s = PD_ERR_DEVICE;
          break;
        }
        ms_per_stage[k] += ms / n_iter;
      }
    if (layer1_unpacks(h, batch, -1)) ms_per_stage[0] = 0.0f;  // no kernel between the first two events
  }
  for (auto& e : ev)
    if (e) (void)hipEventDestroy(e);
  (void)hipGetLastError();
  return s;
}

void predecoder_destroy(pd_predecoder* h) {
  if (!h) return;
  (void)hipDeviceSynchronize();
  free_all(h);
  delete h;
}

pd_status predecoder_graph_create(pd_predecoder* h, const uint64_t* det, int32_t batch, uint64_t* flips,
                                  uint64_t* residual, float* logits, pd_graph** out) {
  if (!out) return PD_ERR_INVALID_ARG;
  *out = nullptr;
  if (!h || !det || !flips || !residual) return PD_ERR_INVALID_ARG;
  if (batch < 1 || batch > h->max_batch) return PD_ERR_INVALID_ARG;
  pd_graph* gr = new (std::nothrow) pd_graph();
  if (!gr) return PD_ERR_OUT_OF_MEMORY;
  auto fail = [&](pd_status e) {
    (void)hipGetLastError();
    if (gr->exec) (void)hipGraphExecDestroy(gr->exec);
    if (gr->graph) (void)hipGraphDestroy(gr->graph);
    if (gr->stream) (void)hipStreamDestroy(gr->stream);
    delete gr;
    return e;
  };
  // a stream of its own at the default priority (capture needs a stream
  // other than the null stream)
  if (hipStreamCreateWithFlags(&gr->stream, hipStreamNonBlocking) != hipSuccess) return fail(PD_ERR_DEVICE);
  // one run first: the handle's buffers reach the state every later run
  // starts from, so the recorded sequence (with any buffer clearing it
  // needs) is the one each replay repeats
  pd_status s = enqueue_run(h, h->ws, gr->stream, det, batch, flips, residual, logits, nullptr);
  if (s != PD_OK) return fail(s);
  if (hipStreamSynchronize(gr->stream) != hipSuccess) return fail(PD_ERR_DEVICE);
  if (hipStreamBeginCapture(gr->stream, hipStreamCaptureModeThreadLocal) != hipSuccess) return fail(PD_ERR_DEVICE);
  s = enqueue_run(h, h->ws, gr->stream, det, batch, flips, residual, logits, nullptr);
  hipGraph_t graph = nullptr;
  const hipError_t ec = hipStreamEndCapture(gr->stream, &graph);
  gr->graph = graph;
  if (s != PD_OK) return fail(s);
  if (ec != hipSuccess || !graph) return fail(PD_ERR_DEVICE);
  if (hipGraphInstantiate(&gr->exec, graph, nullptr, nullptr, 0) != hipSuccess) return fail(PD_ERR_DEVICE);
  *out = gr;
  return PD_OK;
}

pd_status predecoder_graph_launch(pd_graph* gr, void* hip_stream) {
  if (!gr || !gr->exec) return PD_ERR_INVALID_ARG;
  return check_launch(hipGraphLaunch(gr->exec, (hipStream_t)hip_stream));
}

void predecoder_graph_destroy(pd_graph* gr) {
  if (!gr) return;
  (void)hipDeviceSynchronize();
  if (gr->exec) (void)hipGraphExecDestroy(gr->exec);
  if (gr->graph) (void)hipGraphDestroy(gr->graph);
  if (gr->stream) (void)hipStreamDestroy(gr->stream);
  delete gr;
}

int32_t predecoder_stream_windows(int32_t n_rounds, int32_t core, int32_t buffer, int32_t* starts, int32_t* lengths,
                                  int32_t* core_starts, int32_t* core_lengths, int32_t capacity) {
  if (n_rounds < 1 || core < 1 || buffer < 0) return -1;
  const int32_t n = (n_rounds + core - 1) / core;
  if (!starts || !lengths || !core_starts || !core_lengths) return n;
  if (capacity < n) return -1;
  for (int32_t k = 0; k < n; ++k) {
    const int32_t c0 = k * core, c1 = std::min(n_rounds, c0 + core);
    const int32_t w0 = std::max(0, c0 - buffer), w1 = std::min(n_rounds, c1 + buffer);
    starts[k] = w0;
    lengths[k] = w1 - w0;
    core_starts[k] = c0;
    core_lengths[k] = c1 - c0;
  }
  return n;
}

}  // extern "C"

// Temporal window driver: a handle per group of windows (those of one length
// that touch round 0 / the last round alike, or all of them, see
// plan_stream) runs them for all streams as one batch.
struct pd_stream {
  int d = 0, n_rounds = 0, core = 0, buffer = 0, n_streams = 0;
  pd::Geom g;                          // the whole stream (for its residual)
  int32_t* tables = nullptr;           // its site tables
  std::vector<pd::StreamWindow> win;   // host copy
  pd::StreamWindow* win_dev = nullptr;
  struct Group {
    int len = 0, count = 0;
    pd_predecoder* h = nullptr;
    uint64_t *det = nullptr, *flips = nullptr, *res = nullptr;
    pd::StreamWindow* win_dev = nullptr;  // this group's windows, in slot order
  };
  std::vector<Group> groups;
  uint64_t** group_flips_dev = nullptr;
  long long* group_words_dev = nullptr;
};

namespace {
// A plain network's run of `batch` samples as a handle would plan it (no device memory).
struct PlannedRun {
  pd_predecoder h;
  int batch;
};

PlannedRun plan_run(const pd_layer* layers, int dtype, int layout, int d, int T, int batch, int n_cu) {
  PlannedRun r;
  r.h.ks = network_ks(layers);
  r.h.g = make_geom(d, T, layout, 0, 0, (r.h.ks - 1) / 2);
  r.h.dtype = dtype;
  r.h.n_cu = n_cu;
  r.batch = batch;
  if (dtype != PD_DTYPE_FP32) plan_tilings(&r.h, batch);
  return r;
}

// Whether every hidden layer of a plain bf16 network takes its sums in the
// same parts in both runs (no sample apart).  (fp32 sums have one order; fp8
// ones may differ in order between the kernels that two batch sizes run on, as
// predecoder_run's do.)
bool same_sums(const pd_layer* layers, int n, const PlannedRun& a, const PlannedRun& b) {
  if (a.h.dtype != PD_DTYPE_BF16) return true;
  for (int l = 1; l < n - 1; ++l) {
    const LayerRun L = plain_layer(layers, n, l);
    const SumPlan p = sum_plan(&a.h, L, a.batch), q = sum_plan(&b.h, L, b.batch);
    if (p.parts != q.parts || p.first != a.batch || q.first != b.batch) return false;
  }
  return true;
}

// Estimated microseconds of a run: its hidden layers as their launches are
// chosen (small_us, big_us; past a round of units, full rounds and the rest),
// and for the launches around them and the gaps between 50, and 0.4 ns per
// voxel.  (Of 424 streams timed both ways, d = 5 to 31, it takes the slower way by
// more than 5 % in 3.)
double run_us(const pd_layer* layers, int n, const PlannedRun& r) {
  const pd_predecoder& h = r.h;
  double us = 50.0 + 4e-4 * r.batch * h.g.V;
  for (int l = 1; l < n; ++l) {
    if (l == n - 1 && layers[l].k != 5) break;  // (the head, or a 3x3x3 output layer: part of the above)
    const LayerRun L = plain_layer(layers, n, l);
    if (h.dtype == PD_DTYPE_FP32) {
      const pd::Fp32Blocks b = pd::conv_fp32_blocks((long long)r.batch * h.g.V, L.cout, l == n - 2, h.n_cu);
      us += 5.0 + b.cost * (27.0 * L.cin / 16.0) / 2100.0;
      continue;
    }
    Launch q[2];
    const int k = layer_launches(&h, L, r.batch, q);
    for (int i = 0; i < k; ++i) {
      if (q[i].small) {
        us += small_us(&h, L, q[i].nb, q[i].parts, &q[i].plan);
        continue;
      }
      Tiling t = h.tiling;
      tiling_for_batch(&t, h.g, q[i].nb);
      const BigTime bt = big_time(&h, L);
      const long long units = t.ntiles * (L.cout / L.cw), rest = units % bt.round;
      us += units / bt.round * bt.t2 + (rest ? big_us(bt, rest) : 0.0);
    }
  }
  return us;
}

// The batches of a stream: its windows, per batch their length, count and
// whether they touch the stream's first / last round, and the samples whose
// geometric channels are cleared there (Geom::first_n, last_from).
struct StreamPlan {
  struct Batch {
    int len, count, first, last;
  };
  std::vector<pd::StreamWindow> win;
  std::vector<Batch> batches;
  int first_n = INT_MAX, last_from = 0;
};

// n_cu 0: unknown, windows of one length and boundary kind per batch.
StreamPlan plan_stream(const pd_layer* layers, int n_layers, int d, int n_rounds, int core, int buffer, int dtype,
                       int layout, int n_streams, int n_cu) {
  const int nw = predecoder_stream_windows(n_rounds, core, buffer, nullptr, nullptr, nullptr, nullptr, 0);
  std::vector<int32_t> st(nw), ln(nw), cs(nw), cl(nw);
  predecoder_stream_windows(n_rounds, core, buffer, st.data(), ln.data(), cs.data(), cl.data(), nw);
  StreamPlan p;
  // a batch per length, first-round window, last-round window (the paper
  // layout clears its geometric channels only at the stream's own ends)
  p.win.resize(nw);
  for (int k = 0; k < nw; ++k) {
    const int first = st[k] == 0, last = st[k] + ln[k] == n_rounds;
    int b = 0;
    while (b < (int)p.batches.size() &&
           (p.batches[b].len != ln[k] || p.batches[b].first != first || p.batches[b].last != last))
      ++b;
    if (b == (int)p.batches.size()) p.batches.push_back({ln[k], 0, first, last});
    p.win[k] = pd::StreamWindow{st[k], ln[k], cs[k], cl[k], b, p.batches[b].count++};
  }
  // All windows as one batch of the longest window's length: the shorter ones,
  // at the stream's ends, read further rounds that their cores do not depend
  // on (the buffer reaches the receptive field), and the geometric channels
  // are cleared for the first / last windows' samples.  One run then takes
  // the place of up to five, four of them a few windows each (Model 4, d =
  // 13, bf16, two streams of 1000 rounds: 3.36 -> 2.99 ms).  Only where no
  // bf16 sum's parts change, and where the further rounds cost less than the
  // launches saved: a few windows of many streams fill the chip anyway (64
  // streams of 39 rounds, three windows: 3.17 ms in three batches, 3.76 in one
  // of 29 % more rounds).
  int reach = 0;
  for (int l = 0; l < n_layers; ++l) reach += (layers[l].k - 1) / 2;
  if (n_cu < 1 || p.batches.size() < 2 || buffer < reach || !layer_chain_ok(layers, n_layers, layout)) return p;
  const int len = *std::max_element(ln.begin(), ln.end());
  const Geom whole = make_geom(d, len, layout, 0, 0, (network_ks(layers) - 1) / 2);
  if (!supported(whole, layers, n_layers, dtype) || (long long)nw * n_streams * whole.S >= (1ll << 30)) return p;
  const PlannedRun all = plan_run(layers, dtype, layout, d, len, nw * n_streams, n_cu);
  double batches_us = 0.0;
  for (const auto& b : p.batches) {
    const PlannedRun run = plan_run(layers, dtype, layout, d, b.len, b.count * n_streams, n_cu);
    if (!same_sums(layers, n_layers, run, all)) return p;
    batches_us += run_us(layers, n_layers, run);
  }
  if (run_us(layers, n_layers, all) >= batches_us) return p;
  p.batches.assign(1, {len, nw, 1, 1});
  int firsts = 0, lasts = 0;
  for (int k = 0; k < nw; ++k) {
    const int start = std::min(st[k], n_rounds - len);
    firsts += start == 0;
    lasts += start + len == n_rounds;
    p.win[k] = pd::StreamWindow{start, len, cs[k], cl[k], 0, k};
  }
  p.first_n = firsts * n_streams;
  p.last_from = (nw - lasts) * n_streams;
  return p;
}

void stream_free(pd_stream* s) {
  for (auto& g : s->groups) {
    if (g.h) predecoder_destroy(g.h);
    if (g.det) (void)hipFree(g.det);
    if (g.flips) (void)hipFree(g.flips);
    if (g.res) (void)hipFree(g.res);
    if (g.win_dev) (void)hipFree(g.win_dev);
  }
  if (s->tables) (void)hipFree(s->tables);
  if (s->win_dev) (void)hipFree(s->win_dev);
  if (s->group_flips_dev) (void)hipFree(s->group_flips_dev);
  if (s->group_words_dev) (void)hipFree(s->group_words_dev);
  delete s;
}
}  // namespace

extern "C" {

// For the tests: the batches that a stream's windows run in, planned without
// a device for one of n_cu compute units; -1 for arguments without a plan.
int32_t pd_plan_stream(const pd_layer* layers, int32_t n_layers, int32_t d, int32_t n_rounds, int32_t core,
                       int32_t buffer, int32_t dtype, int32_t layout, int32_t n_streams, int32_t n_cu) {
  if (predecoder_stream_windows(n_rounds, core, buffer, nullptr, nullptr, nullptr, nullptr, 0) < 1) return -1;
  return (int32_t)plan_stream(layers, n_layers, d, n_rounds, core, buffer, dtype, layout, n_streams, n_cu)
      .batches.size();
}

// predecoder_stream_create with its arguments checked and its windows planned for n_cu compute units.
static pd_status create_stream(const float* weights, size_t n_weights, int32_t d, int32_t n_rounds, int32_t core,
                               int32_t buffer, const pd_layer* layers, int32_t n_layers, int32_t dtype,
                               int32_t n_streams, const pd_options& o, int n_cu, pd_stream** out) {
  const StreamPlan plan = plan_stream(layers, n_layers, d, n_rounds, core, buffer, dtype, o.layout, n_streams, n_cu);
  pd_stream* s = new (std::nothrow) pd_stream();
  if (!s) return PD_ERR_OUT_OF_MEMORY;
  s->d = d;
  s->n_rounds = n_rounds;
  s->core = core;
  s->buffer = buffer;
  s->n_streams = n_streams;
  s->win = plan.win;
  for (const auto& b : plan.batches) {
    s->groups.emplace_back();
    s->groups.back().len = b.len;
    s->groups.back().count = b.count;
  }
  pd_status r = PD_OK;
  auto fail = [&](pd_status e) {
    stream_free(s);
    return e;
  };
  for (size_t gi = 0; gi < s->groups.size(); ++gi) {
    auto& G = s->groups[gi];
    pd_options go = o;
    if (!plan.batches[gi].first) go.first_round = PD_BOUNDARY_NONE;
    if (!plan.batches[gi].last) go.last_round = PD_BOUNDARY_NONE;
    r = predecoder_create_ex(weights, n_weights, d, G.len, layers, n_layers, dtype, G.count * n_streams, &go, &G.h);
    if (r != PD_OK) return fail(r);
    G.h->g.first_n = plan.first_n;
    G.h->g.last_from = plan.last_from;
    const size_t rows = (size_t)G.count * n_streams;
    if ((r = dev_alloc(&G.det, rows * predecoder_det_words(d, G.len) * 8)) != PD_OK) return fail(r);
    if ((r = dev_alloc(&G.flips, rows * predecoder_flip_words(d, G.len) * 8)) != PD_OK) return fail(r);
    if ((r = dev_alloc(&G.res, rows * predecoder_det_words(d, G.len) * 8)) != PD_OK) return fail(r);
    std::vector<pd::StreamWindow> mine;
    for (const auto& w : s->win)
      if (w.group == (int)gi) mine.push_back(w);
    if ((r = upload(&G.win_dev, mine.data(), mine.size() * sizeof(pd::StreamWindow))) != PD_OK) return fail(r);
  }
  s->g = make_geom(d, n_rounds, o.layout, o.first_round, o.last_round);
  std::vector<int32_t> tab = build_tables(s->g);
  if ((r = upload(&s->tables, tab.data(), tab.size() * sizeof(int32_t))) != PD_OK) return fail(r);
  if ((r = upload(&s->win_dev, s->win.data(), s->win.size() * sizeof(pd::StreamWindow))) != PD_OK) return fail(r);
  std::vector<uint64_t*> gf;
  std::vector<long long> gw;
  for (auto& G : s->groups) {
    gf.push_back(G.flips);
    gw.push_back(predecoder_flip_words(d, G.len));
  }
  if ((r = upload(&s->group_flips_dev, gf.data(), gf.size() * sizeof(uint64_t*))) != PD_OK) return fail(r);
  if ((r = upload(&s->group_words_dev, gw.data(), gw.size() * sizeof(long long))) != PD_OK) return fail(r);
  if (hipDeviceSynchronize() != hipSuccess) return fail(PD_ERR_DEVICE);
  *out = s;
  return PD_OK;
}

pd_status predecoder_stream_create(const float* weights, size_t n_weights, int32_t d, int32_t n_rounds, int32_t core,
                                   int32_t buffer, const pd_layer* layers, int32_t n_layers, int32_t dtype,
                                   int32_t n_streams, const pd_options* opts, pd_stream** out) {
  if (!out) return PD_ERR_INVALID_ARG;
  *out = nullptr;
  if (!weights || !layers || n_rounds < 1 || core < 1 || buffer < 0 || n_streams < 1) return PD_ERR_INVALID_ARG;
  if (d < 3 || d % 2 == 0 || n_rounds > kMaxT) return d < 3 || d % 2 == 0 ? PD_ERR_INVALID_ARG : PD_ERR_UNSUPPORTED;
  const pd_options o = opts ? *opts : pd_options{PD_LAYOUT_PLAQUETTE, PD_BOUNDARY_NONE, PD_BOUNDARY_NONE};
  const int32_t nw = predecoder_stream_windows(n_rounds, core, buffer, nullptr, nullptr, nullptr, nullptr, 0);
  if (nw < 1) return PD_ERR_INVALID_ARG;
  int n_cu = 0, dev = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    n_cu = 0;
  (void)hipGetLastError();
  pd_status r = create_stream(weights, n_weights, d, n_rounds, core, buffer, layers, n_layers, dtype, n_streams, o,
                              n_cu, out);
  // (one batch needs a little more memory than several)
  if (r == PD_ERR_OUT_OF_MEMORY && n_cu > 0)
    r = create_stream(weights, n_weights, d, n_rounds, core, buffer, layers, n_layers, dtype, n_streams, o, 0, out);
  return r;
}

pd_status predecoder_stream_run(pd_stream* s, void* hip_stream, const uint64_t* det, uint64_t* flips,
                                uint64_t* residual) {
  if (!s || !det || !flips || !residual) return PD_ERR_INVALID_ARG;
  const hipStream_t st = (hipStream_t)hip_stream;
  const int S = s->d * s->d - 1, F = 3 * s->d * s->d - 1;
  const long long det_words = predecoder_det_words(s->d, s->n_rounds);
  const long long flip_words = predecoder_flip_words(s->d, s->n_rounds);
  pd_status r;
  for (auto& G : s->groups) {
    r = check_launch(pd::launch_stream_gather(det, det_words, G.win_dev, G.count, s->n_streams, S,
                                              predecoder_det_words(s->d, G.len), G.det, st));
    if (r != PD_OK) return r;
    r = predecoder_run(G.h, hip_stream, G.det, G.count * s->n_streams, G.flips, G.res, nullptr);
    if (r != PD_OK) return r;
  }
  r = check_launch(pd::launch_stream_scatter(s->win_dev, s->group_flips_dev, s->group_words_dev, s->n_streams,
                                             s->core, s->n_rounds, F, flip_words, flips, st));
  if (r != PD_OK) return r;
  return check_launch(pd::launch_residual_from_flips(s->g, s->tables, det, flips, residual, s->n_streams, st));
}

void predecoder_stream_destroy(pd_stream* s) {
  if (!s) return;
  (void)hipDeviceSynchronize();
  stream_free(s);
}

}  // extern "C"
