"""The launches that the library plans for a network, asked of its host code (no GPU)."""
import collections
import ctypes

import paper_2604_12841_amd as pdx

# layer: of a plain network, or conv1 / conv2 of block k as 2 k / 2 k + 1; rows, cols: voxels and channels of a tile
# (256 voxels: the persistent kernel; fp32: of a wave); parts: K parts of a sum; counters: units come from counters
Launch = collections.namedtuple("Launch", "layer samples rows cols parts counters")


def launches(d, T, dtype, batch, layers=None, blocks=None, layout="plaquette", max_batch=None, n_cu=256):
    out = (ctypes.c_int32 * 1200)()
    n = pdx.lib().pd_plan_launches(
        pdx._layers(layers) if layers else None, len(layers or ()), pdx._blocks(blocks) if blocks else None,
        len(blocks or ()), d, T, pdx._DTYPES[dtype], pdx._LAYOUTS[layout], batch, max_batch or batch, n_cu, out, 200)
    assert 0 <= n <= 200, n
    return [Launch(*out[6 * k:6 * k + 6]) for k in range(n)]


def network(layout, widths, k=3, act=1):
    layers, ci = [], 2 if layout == "plaquette" else 4
    for w in widths:
        layers.append((ci, w, k, act))
        ci = w
    return layers + [(ci, 4, 1 if layout == "plaquette" else k, 0)]


def stream_batches(layers, d, n_rounds, core, buffer, dtype, n_streams, layout="paper", n_cu=256):
    """Batches that a stream's windows run in."""
    return pdx.lib().pd_plan_stream(pdx._layers(layers), len(layers), d, n_rounds, core, buffer, pdx._DTYPES[dtype],
                                    pdx._LAYOUTS[layout], n_streams, n_cu)


def small_instances(d, T, dtype, batch, layers=None, blocks=None, layout="plaquette"):
    """Instances of the small-launch kernel that a network's launches run: (dtype, kernel size, pieces of an input row
    (half, one, more), voxels, channels, parts of a sum (fp8: 0, over 4: 8, over 16: 32), epilogue)."""
    out = set()
    for r in launches(d, T, dtype, batch, layers, blocks, layout):
        if r.rows == 256:
            continue
        if blocks:
            ci, ks, epi = blocks[r.layer // 2][r.layer % 2], 3, "add" if r.layer % 2 else "act"
        else:
            ci, co, ks = layers[r.layer][:3]
            head = layers[-1][2] == 1 and r.layer == len(layers) - 2
            epi = "out" if r.layer == len(layers) - 1 else "head" if head and co == 64 else "act"
        row = ci * (1 if dtype == "fp8" else 2)
        parts = 0 if dtype == "fp8" else r.parts if r.parts <= 4 else 8 if r.parts <= 16 else 32
        out.add((dtype, ks, "half" if row < 128 else "one" if row == 128 else "more", r.rows, r.cols, parts, epi))
    return out
