// tiles.h -- output-row tiles of the 3x3x3 conv kernels (tile -> rows, the
// staged input footprint, the XCD-aware tile order).  See Tiling in
// internal.h for the two modes.
#pragma once

#include "internal.h"

namespace pd {

// Cell-mode (mode 1) tile: its sample, run number within the cell, and the
// cell's first grid row and column.
struct CellTile {
  int b, run, i0, j0;
};

__host__ __device__ inline CellTile cell_tile(const Tiling& tl, int tile) {
  const int per = tl.ntT * tl.ntI * tl.ntJ, ntij = tl.ntI * tl.ntJ;
  CellTile ct;
  ct.b = (int)fdiv((uint32_t)tile, tl.dv_per);
  const int rem = tile - ct.b * per;
  ct.run = (int)fdiv((uint32_t)rem, tl.dv_ntij);
  const int rem2 = rem - ct.run * ntij;
  const int ti = (int)fdiv((uint32_t)rem2, tl.dv_ntj);
  ct.i0 = ti * tl.BI;
  ct.j0 = (rem2 - ti * tl.ntJ) * tl.BJ;
  return ct;
}

// Voxel u of a cell, in (t, i, j) order (of any tile size): its round, row and column in the cell.
__host__ __device__ inline void cell_voxel(const Tiling& tl, int u, int* a, int* c, int* e) {
  const int bij = tl.BI * tl.BJ;
  *a = (int)fdiv((uint32_t)u, tl.dv_bij);
  const int r = u - *a * bij;
  *c = (int)fdiv((uint32_t)r, tl.dv_bj);
  *e = r - *c * tl.BJ;
}

// Row r (0..255) of tile `tile`: false if the row is outside the volume,
// else its padded output index (pidx) and its column j (col).  Also the LDS
// voxel of the row's (0,0,0) tap (lds_base) and the staging origin: the
// line-space index of staged voxel 0 (mode 0) or its padded index (mode 1).
// 32-bit voxel counts: the host guarantees max_batch * V < 2^31.  Divisions
// by the run-time sizes use the Tiling's precomputed multipliers (a plain
// integer division costs tens of instructions per lane, which small
// batches, with one tile per workgroup, pay in full).
__host__ __device__ inline bool tile_row(const Geom& g, const Tiling& tl, int tile, int r, int batch,
                                         long long* pidx, int* lds_base, long long* stage_origin,
                                         int* col = nullptr) {
  const int HH = g.H * g.H;
  if (tl.mode == 0) {
    const int seg = (int)fdiv((uint32_t)tile, tl.dv_tps);
    const int k0 = (tile - seg * tl.tiles_per_seg) * kTileRows;
    const int u0 = seg * (int)tl.seg_len + k0;
    const int b0 = (int)fdiv((uint32_t)u0, tl.dv_V);
    const int v0 = u0 - b0 * g.V;
    const int t0 = (int)fdiv((uint32_t)v0, tl.dv_HH), s0 = v0 - t0 * HH;
    const int i0 = (int)fdiv((uint32_t)s0, tl.dv_H);
    const long long l0 = line_index(g, b0, t0, i0, s0 - i0 * g.H);
    *stage_origin = l0 - (line_plane(g) + g.H + 1);
    const int u = u0 + r;
    if (k0 + r >= tl.seg_len || u >= batch * g.V) {
      *lds_base = 0;
      if (col) *col = -1;
      return false;
    }
    const int b = (int)fdiv((uint32_t)u, tl.dv_V);
    const int v = u - b * g.V;
    const int t = (int)fdiv((uint32_t)v, tl.dv_HH), s = v - t * HH;
    const int i = (int)fdiv((uint32_t)s, tl.dv_H), j = s - i * g.H;
    *pidx = padded_index(g, b, t, i, j);
    *lds_base = (int)(line_index(g, b, t, i, j) - l0);
    if (col) *col = j;
    return true;
  } else {
    const CellTile ct = cell_tile(tl, tile);
    int a0, c0, e0, a, c, e;
    cell_voxel(tl, ct.run * kTileRows, &a0, &c0, &e0);
    *stage_origin = (long long)ct.b * g.S + (long long)a0 * g.P + (long long)(ct.i0 + c0) * g.Wp + ct.j0 + e0;
    cell_voxel(tl, ct.run * kTileRows + r, &a, &c, &e);
    const int i = ct.i0 + c, j = ct.j0 + e;
    const bool ok = a < g.T && i < g.H && j < g.H;
    *lds_base = ok ? (a - a0) * tl.sa + (c - c0) * tl.sb + e - e0 : 0;
    if (col) *col = ok ? j : -1;
    if (!ok) return false;
    *pidx = padded_index(g, ct.b, a, i, j);
    return true;
  }
}

// Sample and grid coordinates (b, t, i, j) of row r of tile `tile`; false if
// the row is outside the volume.  32-bit arithmetic (max_batch * V < 2^31).
__host__ __device__ inline bool tile_row_coords(const Geom& g, const Tiling& tl, int tile, int r, int batch,
                                                int* b, int* t, int* i, int* j) {
  const int HH = g.H * g.H;
  if (tl.mode == 0) {
    const int seg = (int)fdiv((uint32_t)tile, tl.dv_tps);
    const int k0 = (tile - seg * tl.tiles_per_seg) * kTileRows;
    const int u = seg * (int)tl.seg_len + k0 + r;
    if (k0 + r >= tl.seg_len || u >= batch * g.V) return false;
    *b = (int)fdiv((uint32_t)u, tl.dv_V);
    const int v = u - *b * g.V;
    *t = (int)fdiv((uint32_t)v, tl.dv_HH);
    const int s = v - *t * HH;
    *i = (int)fdiv((uint32_t)s, tl.dv_H);
    *j = s - *i * g.H;
    return true;
  }
  const CellTile ct = cell_tile(tl, tile);
  int c, e;
  cell_voxel(tl, ct.run * kTileRows + r, t, &c, &e);
  *b = ct.b;
  *i = ct.i0 + c;
  *j = ct.j0 + e;
  return *t < g.T && *i < g.H && *j < g.H;
}

// Tile handled by persistent workgroup `wg` at iteration `it`: the 8 XCDs
// receive workgroups round-robin, so workgroup wg runs on XCD wg % 8; each
// XCD gets a contiguous range of tiles (neighbouring tiles share halo voxels
// in its L2) and its workgroups stride through it.  -1 when done.
__host__ __device__ inline int tile_of(int wg, int nwg, int it, int ntiles) {
  const int xcd = wg & 7, k = wg >> 3, per_xcd_wg = nwg >> 3;
  const int per_xcd = (ntiles + 7) >> 3;
  const int idx = k + it * per_xcd_wg;
  if (idx >= per_xcd) return -1;
  const int t = xcd * per_xcd + idx;
  return t < ntiles ? t : -1;
}

// Staging source of a tile: the origin (see tile_row), and in mode 1 the
// line index of staged voxel 0 in the cell's padded line space, the cell's
// first row and column, and what to add to a line's decoded a P + c Wp + e to
// count from the origin.
struct StageSrc {
  long long origin;
  int line0, i0, j0, back;
};

__host__ __device__ inline StageSrc tile_source(const Geom& g, const Tiling& tl, int tile, int batch) {
  StageSrc src{0, 0, 0, 0, 0};
  if (tl.mode == 0) {
    long long p;
    int lb;
    tile_row(g, tl, tile, 0, batch, &p, &lb, &src.origin);
  } else {
    const CellTile ct = cell_tile(tl, tile);
    int a0, c0, e0;
    cell_voxel(tl, ct.run * kTileRows, &a0, &c0, &e0);
    const int first = a0 * g.P + c0 * g.Wp + e0;
    src.origin = (long long)ct.b * g.S + first + (long long)ct.i0 * g.Wp + ct.j0;
    src.line0 = a0 * tl.sa + c0 * tl.sb + e0;
    src.i0 = ct.i0;
    src.j0 = ct.j0;
    src.back = -first;
  }
  return src;
}

// Global padded voxel of staged voxel vv; -1 when it is outside the batch or
// the sample's padded box (such voxels only feed rows that are discarded).
template <int MODE>
__host__ __device__ inline long long staged_voxel(const Geom& g, const Tiling& tl, const StageSrc& src, int vv,
                                                  long long limit) {
  if constexpr (MODE == 0) {
    const uint32_t u = (uint32_t)(src.origin + vv);  // < 2^31 (host check)
    const uint32_t tp = fastdiv(u, tl.div_a);
    const uint32_t rem = u - tp * (uint32_t)tl.sa;
    const uint32_t ip = fastdiv(rem, tl.div_b);
    const uint32_t jj = rem - ip * (uint32_t)g.H;
    const long long p = (long long)tp * g.P + (long long)ip * g.Wp + jj + 1;
    return p < limit ? p : -1;
  } else {
    const int u = src.line0 + vv;
    const int a = (int)fastdiv((uint32_t)u, tl.div_a);
    const int rem = u - a * tl.sa;
    const int c = (int)fastdiv((uint32_t)rem, tl.div_b);
    const int e = rem - c * tl.sb;
    if (a >= g.T + 2 * g.pad || src.i0 + c >= g.Wp || src.j0 + e >= g.Wp) return -1;
    return src.origin + (a * g.P + c * g.Wp + e + src.back);
  }
}

}  // namespace pd
