"""Per-layer checks of the small-launch conv kernel and of cell tilings.

Every hidden layer's stored activations are recomputed in fp64 from the GPU's
own input (the planes, then what the GPU stored for the layer before) under
the rule of tests/tight.py, whose bounds hold for any order of a sum's parts.
The networks and batches reach every instance of the kernel that the choice of
launches takes (tests/test_launch_plan.py checks that they do): its K parts, tile
shapes and epilogues, input rows of half a piece to four pieces, 3x3x3 and 5x5x5
layers, on one-round and ragged grids; CASES holds at last some of the persistent kernel
on cells whose tiles start and end inside a round."""
import numpy as np
import pytest

import paper_2604_12841_amd as pdx
import test_gpu_model6 as resnets
import test_gpu_model6_fp8 as resnets_fp8
import tight
from paper_2604_12841_amd import workload
from parity import dev_u64, say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

G, R, N = workload.GELU_TANH, workload.RELU, workload.NONE


@pytest.fixture(scope="module")
def cuda():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda")


def network(layout, widths, k=3, act=G):
    layers, ci = [], 2 if layout == "plaquette" else 4
    for w in widths:
        layers.append((ci, w, k, act))
        ci = w
    layers.append((ci, 4, 1 if layout == "plaquette" else k, N))
    return layers


def quantised(w, dtype):
    """Weights [c_out][...] at the handle's precision."""
    if dtype == "bf16":
        return tight.q_bf16(w)
    amax = w.flatten(1).abs().amax(1)
    e = torch.ceil(torch.log2(amax / 448.0))
    e = torch.where(amax / torch.exp2(e - 1) <= 448.0, e - 1, e)
    s = torch.exp2(e).view(-1, 1, 1, 1, 1)
    return tight.q_e4m3(w / s) * s


CASES = [
    # layout, hidden widths, k, d, T, B, dtype
    ("plaquette", [64, 64, 64], 3, 5, 5, 1, "bf16"),        # four parts of one chunk
    ("plaquette", [128, 128, 128], 3, 5, 1, 1, "bf16"),     # eight parts, one round of syndrome
    ("plaquette", [128, 128, 128], 3, 13, 13, 1, "bf16"),   # four parts
    ("plaquette", [128, 64, 128], 3, 17, 17, 1, "bf16"),    # four parts, then one; mixed widths
    ("plaquette", [64, 64, 64], 3, 21, 9, 2, "bf16"),       # one part, 64-channel head in the tile
    ("plaquette", [128, 128, 128], 3, 25, 14, 1, "bf16"),   # one part, 128-channel head after the layer
    ("plaquette", [64, 64], 3, 63, 3, 1, "bf16"),           # the widest grid
    ("plaquette", [64, 64, 64], 3, 3, 2, 1, "fp8"),         # half a piece per voxel
    ("plaquette", [128, 128, 64], 3, 13, 13, 1, "fp8"),
    ("plaquette", [128, 128, 128], 3, 21, 7, 3, "fp8"),
    ("paper", [256, 256, 256], 3, 7, 5, 1, "bf16"),         # sixteen parts, four pieces
    ("paper", [256, 256, 256], 3, 13, 13, 1, "bf16"),       # eight parts
    ("paper", [256, 256, 64], 3, 17, 12, 1, "bf16"),
    ("paper", [256, 256, 256], 3, 13, 9, 1, "fp8"),         # two pieces
    ("paper", [128, 256, 128], 3, 11, 4, 1, "fp8"),
    ("paper", [64, 64, 64], 5, 5, 4, 1, "bf16"),            # 5x5x5, one piece
    ("paper", [128, 128, 128], 5, 9, 9, 1, "bf16"),         # ... eight parts
    ("paper", [128, 128], 5, 13, 6, 3, "bf16"),
    # the other instances, the smallest launches that reach them: 64-channel heads in the tile, by parts and tiles
    ("plaquette", [128, 128, 64], 3, 3, 1, 36, "bf16"),
    ("plaquette", [128, 128, 64], 3, 3, 2, 72, "bf16"),
    ("plaquette", [128, 128, 64], 3, 3, 2, 250, "bf16"),
    ("plaquette", [128, 128, 64], 3, 3, 5, 150, "bf16"),
    ("plaquette", [128, 128, 64], 3, 3, 1, 72, "bf16"),
    ("plaquette", [128, 128, 64], 3, 5, 2, 150, "bf16"),
    ("plaquette", [64, 64, 64], 3, 3, 5, 150, "bf16"),
    ("paper", [64, 256], 3, 3, 1, 250, "bf16"),
    # fp8 128 x 64 tiles (a wide grid of one round)
    ("plaquette", [64, 64, 64], 3, 43, 1, 16, "fp8"),
    ("plaquette", [128, 128, 64], 3, 43, 1, 16, "fp8"),
    # 5x5x5 layers of one piece, and of two
    ("paper", [64, 64], 5, 3, 1, 72, "bf16"),
    ("paper", [64, 64], 5, 3, 1, 150, "bf16"),
    ("paper", [64, 64], 5, 5, 3, 72, "bf16"),
    ("paper", [64, 64], 5, 5, 3, 150, "bf16"),
    ("paper", [64, 64], 5, 11, 1, 48, "bf16"),
    ("paper", [64, 64], 5, 11, 1, 100, "bf16"),
    ("paper", [64, 64], 5, 21, 2, 16, "bf16"),
    ("paper", [128, 128], 5, 3, 1, 36, "bf16"),
    ("paper", [128, 128], 5, 3, 1, 72, "bf16"),
    ("paper", [128, 128], 5, 3, 1, 150, "bf16"),
    ("paper", [128, 128], 5, 5, 3, 36, "bf16"),
    ("paper", [128, 128], 5, 5, 3, 150, "bf16"),
    ("paper", [128, 128], 5, 11, 1, 24, "bf16"),
    ("paper", [128, 128], 5, 11, 1, 36, "bf16"),
    # 96-voxel tiles of two parts
    ("paper", [128, 128, 128], 5, 13, 13, 8, "bf16"),
    ("paper", [128, 128], 5, 9, 7, 24, "bf16"),
    ("paper", [128, 256, 128], 3, 17, 17, 4, "bf16"),
    # ... and of four parts: one round of the syndrome, a ragged last tile
    ("paper", [256, 256], 3, 17, 1, 11, "bf16"),
    ("paper", [256, 256], 3, 13, 13, 2, "bf16"),
    # the persistent kernel on cells
    ("plaquette", [64, 64], 3, 19, 19, 70, "bf16"),
    ("plaquette", [128, 128], 3, 21, 5, 200, "bf16"),
    ("paper", [128, 128], 3, 29, 6, 80, "fp8"),
]


@pytest.mark.parametrize("layout,widths,k,d,T,B,dtype", CASES,
                         ids=["%s_%s_k%d_d%d_T%d_B%d_%s" % (c[0], "x".join(map(str, c[1])), *c[2:]) for c in CASES])
def test_layers_tight(cuda, layout, widths, k, d, T, B, dtype):
    act = R if T % 2 == 0 else G
    layers = network(layout, widths, k, act)
    weights = workload.he_normal_weights(layers, 301 + d)
    det, _ = workload.make_inputs(d, T, B, 0.03, 0.03, 302)
    basis = "Z" if layout == "paper" else None
    say(layout, widths, "k", k, "d", d, "T", T, "B", B, dtype)
    pre = pdx.Predecoder(weights, d, T, layers, dtype, max_batch=B, layout=layout, first=basis, last=basis)
    ddet, H = dev_u64(det), pre.grid
    pick = sorted({0, B - 1})
    planes = torch.empty((B, T, H, H, layers[0][0]), dtype=torch.int16, device="cuda")
    pre.unpack(ddet, planes)
    torch.cuda.synchronize()
    x = tight.bf16_bits_to_double(planes[pick].cpu()).permute(0, 4, 1, 2, 3).contiguous()
    q = tight.q_bf16 if dtype == "bf16" else tight.q_e4m3
    off = 0
    for l, (ci, co, kk, a) in enumerate(layers[:-1]):
        nw = co * ci * kk ** 3
        w = quantised(torch.from_numpy(weights[off:off + nw].reshape(co, ci, kk, kk, kk).astype(np.float64)), dtype)
        b = torch.from_numpy(weights[off + nw:off + nw + co].astype(np.float64))
        off += nw + co
        y = tight.conv(x, w, b, kk)
        e = tight.eps_bf16_mfma(ci * kk ** 3) if dtype == "bf16" else (2.0 ** -17 if l == 0 else 2.0 ** -16 + 2.0 ** -18)
        eps = e * tight.conv_mag(x, w, b, kk) + tight.U32 * y.abs()
        out = torch.full((B, T, H, H, co), 0x7f, dtype=torch.uint8 if dtype == "fp8" else torch.int16, device="cuda")
        pre.activations(ddet, l, out)
        torch.cuda.synchronize()
        got = out[pick].cpu()
        got = got.view(torch.float8_e4m3fn).double() if dtype == "fp8" else tight.bf16_bits_to_double(got)
        x = got.permute(0, 4, 1, 2, 3).contiguous()
        tight.check_stored("layer %d" % (l + 1), x, y, eps, a, q, say=say)
    # the whole run: the same activations, then the head or output layer, within its own sums' bound
    (ci, co, kk, _), nw = layers[-1], weights.size - off - 4
    w = quantised(torch.from_numpy(weights[off:off + nw].reshape(co, ci, kk, kk, kk).astype(np.float64)), dtype)
    b = torch.from_numpy(weights[off + nw:].astype(np.float64))
    y = tight.conv(x, w, b, kk)
    e = tight.eps_bf16_mfma(ci * kk ** 3) if dtype == "bf16" and kk > 1 else (
        tight.eps_fma_chain(ci) if kk == 1 else 2.0 ** -16 + 2.0 ** -18)
    eps = e * tight.conv_mag(x, w, b, kk) + tight.U32 * y.abs() + 1e-6
    flips = torch.empty((B, pre.flip_words), dtype=torch.int64, device="cuda")
    res = torch.empty((B, pre.det_words), dtype=torch.int64, device="cuda")
    logits = torch.full((B, 4, T, H, H), float("nan"), device="cuda")
    pre.run(ddet, flips, res, logits)
    torch.cuda.synchronize()
    err = (logits[pick].cpu().double() - y).abs()
    say("  logits: max err / bound %.3f" % float((err / eps).max()))
    assert bool((err <= eps).all())
    assert bool(torch.isfinite(logits).all())
    pre.close()


def _resnet(widths, d, T, B, dtype):
    blocks, ci = [], 4
    for w in widths:
        blocks.append((ci, w, w, G))
        ci = w
    blocks.append((ci, ci, 4, G))
    return dict(name="w%s_d%d_T%d_B%d_%s" % ("_".join(map(str, widths)), d, T, B, dtype), blocks=blocks, d=d, T=T, B=B,
                layout="paper", dtype=dtype)


# Layers with a shortcut, and a widening block's first (two parts of one piece)
SHORTCUT_CASES = [_resnet(*c) for c in [
    ([64, 128], 3, 1, 72, "bf16"), ([64, 128], 3, 5, 400, "bf16"), ([64, 128], 9, 1, 72, "bf16"),
    ([64, 128], 43, 1, 4, "bf16"),
    ([128, 64], 5, 3, 250, "bf16"), ([128, 64], 3, 1, 36, "bf16"), ([128, 64], 3, 1, 150, "bf16"),
    ([128, 64], 3, 3, 72, "bf16"), ([128, 64], 9, 1, 36, "bf16"), ([128, 64], 9, 1, 150, "bf16"),
    ([64], 3, 3, 150, "bf16"), ([256], 9, 1, 150, "bf16"),
    ([256], 13, 2, 11, "bf16"), ([512], 9, 2, 11, "bf16"),
    ([64], 3, 1, 400, "fp8"), ([64], 43, 1, 16, "fp8"), ([128], 3, 1, 1, "fp8"), ([128], 3, 1, 150, "fp8"),
    ([128], 43, 1, 8, "fp8"), ([256], 5, 3, 36, "fp8"),
]]


@pytest.mark.parametrize("case", SHORTCUT_CASES, ids=[c["name"] for c in SHORTCUT_CASES])
def test_shortcut_layers_tight(cuda, case):
    (resnets.test_resnet_convs_tight if case["dtype"] == "bf16" else resnets_fp8.test_resnet_fp8_convs_tight)(cuda, case)


def test_resnet_96_voxel_tiles(cuda):
    """Two-part layers with a shortcut (its row, or its projection) in the epilogue."""
    resnets.test_resnet_convs_tight(cuda, dict(name="w128_two_parts", blocks=workload.resnet_blocks([128, 128]), d=9,
                                               T=9, B=24, layout="paper"))


@pytest.mark.parametrize("dtype,B,unpacks", [("bf16", 1, False), ("fp8", 2, False), ("bf16", 128, True), ("fp32", 1, True)])
def test_unpack_stage(cuda, dtype, B, unpacks):
    """Stage 0 takes no time exactly where layer 1 reads the packed events itself."""
    d = 9
    layers = network("plaquette", [64, 64])
    pre = pdx.Predecoder(workload.he_normal_weights(layers, 1), d, d, layers, dtype, max_batch=B)
    det = dev_u64(workload.make_inputs(d, d, B, 0.02, 0.02, 2)[0])
    flips = torch.empty((B, pre.flip_words), dtype=torch.int64, device="cuda")
    res = torch.empty((B, pre.det_words), dtype=torch.int64, device="cuda")
    ms = pre.stage_times(det, flips, res, 3)
    assert (ms[0] > 0) == unpacks and all(t > 0 for t in ms[1:3]), ms
    pre.close()
