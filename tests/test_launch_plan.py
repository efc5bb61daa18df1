"""CPU: the launches planned for the conv layers."""
import ctypes

import pytest

import paper_2604_12841_amd as pdx
from launch_plan import launches, network, small_instances, stream_batches
from paper_2604_12841_amd import workload

NETS = [("plaquette", network("plaquette", w), None, ("bf16", "fp8")) for w in ([64, 64, 64], [128, 128, 128],
                                                                               [64, 128, 64], [128, 64, 128])]
NETS += [("paper", network("paper", w), None, ("bf16", "fp8")) for w in ([128, 128], [256, 256, 256], [256, 256, 64])]
NETS += [("paper", network("paper", [w, w], 5), None, ("bf16",)) for w in (64, 128)]
NETS += [("paper", None, workload.resnet_blocks([w, w]), ("bf16", "fp8")) for w in (64, 128, 256, 512)]


@pytest.mark.parametrize("net", NETS, ids=lambda n: "%s_%s" % (n[0], "x".join(str(l[1]) for l in n[1] or n[2])))
def test_every_launch_has_a_tile(net):
    """Samples add up, a tile's channels divide its slice, and some tile fits every grid and batch."""
    layout, layers, blocks, dtypes = net
    for dtype in dtypes:
        for d in (3, 5, 9, 13, 21, 31, 63):
            for T in (1, 2, 7, d, 1023):
                for batch in (1, 2, 3, 7, 16, 50, 200):
                    if batch > 1 and batch * T * d * d > 1 << 18:
                        break
                    plan = launches(d, T, dtype, batch, layers, blocks, layout)
                    done = {}
                    for r in plan:
                        assert r.rows in (64, 96, 128, 256) and r.cols in (32, 64, 128) and r.parts >= 1, r
                        assert dtype == "fp8" or r.rows < 256 or r.parts == 1, r
                        done[r.layer] = done.get(r.layer, 0) + r.samples
                    assert done and set(done.values()) == {batch}


def test_fp32_blocks_cover_the_head():
    for w in (8, 16, 40, 64, 72, 104, 128):
        for batch in (1, 10, 100, 1000):
            last = launches(5, 5, "fp32", batch, network("plaquette", [32, w]))[-1]
            assert last.cols == (w + 15) // 16 * 16 and last.rows in (16, 32, 64)


def test_short_launches_take_fixed_shares():
    """Up to six units per workgroup (512 workgroups); 64 and 140 samples are 1100 and 1203 units."""
    def counters(model, batch, dtype):
        layers = workload.paper_model_layers(model)
        return {r.counters for r in launches(13, 13, dtype, batch, layers, layout="paper") if r.rows == 256}

    assert counters(5, 64, "bf16") == {0} and counters(4, 140, "fp8") == {0} and counters(4, 330, "bf16") == {0}
    assert counters(5, 200, "bf16") == {1} and counters(4, 4096, "fp8") == {1}


# Networks timed both ways (us: small-launch kernel / persistent kernel), well apart
TIMED = [
    ("w128", "bf16", 13, 37, 323, 273), ("w128", "bf16", 9, 94, 311, 265), ("w128", "bf16", 25, 6, 355, 287),
    ("w128", "bf16", 13, 12, 122, 152), ("w128", "fp8", 13, 12, 83, 100),
    ("w64", "bf16", 5, 718, 151, 129), ("w64", "bf16", 5, 171, 55, 65), ("w64", "fp8", 11, 60, 87, 71),
    ("model2", "fp8", 11, 32, 234, 204), ("model2", "fp8", 7, 138, 255, 208), ("model2", "bf16", 13, 22, 425, 362),
    ("model2", "fp8", 7, 45, 113, 127),
    ("r512", "fp8", 13, 10, 495, 414), ("r512", "fp8", 7, 69, 480, 401), ("r512", "fp8", 17, 4, 543, 421),
    ("r512", "bf16", 11, 20, 892, 766), ("r512", "bf16", 13, 6, 489, 436), ("r512", "fp8", 5, 61, 205, 252),
    ("r128", "bf16", 13, 38, 490, 426), ("r128", "fp8", 7, 119, 161, 199),
]


@pytest.mark.parametrize("net,dtype,d,batch,small,persistent", TIMED, ids=lambda v: str(v))
def test_the_faster_kernel_runs(net, dtype, d, batch, small, persistent):
    layers = {"w128": network("plaquette", [128] * 4), "w64": network("plaquette", [64] * 4),
              "model2": workload.paper_model_layers(2)}.get(net)
    blocks = {"r512": workload.resnet_blocks([512] * 2), "r128": workload.resnet_blocks([128] * 3)}.get(net)
    plan = launches(d, d, dtype, batch, layers, blocks, "plaquette" if net[0] == "w" else "paper")
    assert {r.rows == 256 for r in plan if r.samples > batch // 2} == {persistent < small}, plan


# Layers of four parts timed in their tiles (us: 64 x 32, 64 x 64, 128 x 32, 96 x 64)
TILES = [("model6", 13, 1, 417, 445, 407, 288), ("model5", 5, 64, 228, 190, 271, 225), ("model5", 13, 2, 168, 171, 171, 122),
         ("model2", 17, 1, 96, 99, 99, 77), ("model2", 15, 2, 105, 98, 102, 112), ("r512", 5, 24, 165, 177, 181, 196),
         ("r512", 7, 8, 171, 182, 177, 145), ("model5", 11, 4, 161, 168, 187, 145), ("model5", 7, 16, 165, 170, 176, 169)]


@pytest.mark.parametrize("net,d,batch,t64x32,t64x64,t128x32,t96x64", TILES, ids=lambda v: str(v))
def test_the_fastest_tile_runs(net, d, batch, t64x32, t64x64, t128x32, t96x64):
    layers = {"model2": workload.paper_model_layers(2), "model5": workload.paper_model_layers(5)}.get(net)
    blocks = {"model6": workload.resnet_blocks([512] * 4), "r512": workload.resnet_blocks([512] * 2)}.get(net)
    times = {(64, 32): t64x32, (64, 64): t64x64, (128, 32): t128x32, (96, 64): t96x64}
    plan = launches(d, d, "bf16", batch, layers, blocks, "paper")
    assert {(r.rows, r.cols, r.parts) for r in plan} == {min(times, key=times.get) + (4,)}, plan


# Streams timed both ways, core = buffer = d (us: one batch / a batch per length and boundary kind)
STREAMS = [
    (1, "fp8", 13, 39, 4, 146, 190), (1, "bf16", 13, 39, 8, 327, 402), (4, "bf16", 13, 65, 8, 920, 1165),
    (4, "fp8", 13, 100, 8, 764, 1045), (1, "fp8", 5, 200, 1, 55, 180), (1, "bf16", 21, 150, 1, 428, 548),
    (4, "bf16", 13, 39, 64, 3765, 3174), (4, "bf16", 21, 50, 16, 3227, 2849), (4, "fp8", 21, 50, 16, 1809, 1664),
    (1, "bf16", 31, 93, 2, 931, 857), (4, "bf16", 31, 93, 16, 12817, 10228), (4, "fp8", 31, 93, 16, 7140, 5632),
]


@pytest.mark.parametrize("model,dtype,d,rounds,streams,merged,batches", STREAMS, ids=lambda v: str(v))
def test_stream_windows_merge_where_it_is_faster(model, dtype, d, rounds, streams, merged, batches):
    got = stream_batches(workload.paper_model_layers(model), d, rounds, d, d, dtype, streams)
    assert (got == 1) == (merged < batches), got


def test_stream_windows_that_do_not_merge():
    """A buffer below the receptive field (5 of Model 4), no device, windows that are all alike."""
    layers = workload.paper_model_layers(4)
    assert stream_batches(layers, 13, 1000, 13, 13, "bf16", 2) == 1
    assert stream_batches(layers, 13, 1000, 13, 5, "bf16", 2) > 1
    assert stream_batches(layers, 13, 1000, 13, 13, "bf16", 2, n_cu=0) == 5
    assert stream_batches(layers, 13, 13, 13, 13, "bf16", 2) == 1
    assert stream_batches(layers, 13, 0, 13, 13, "bf16", 2) == -1


def test_head_threads_fit_32_bits():
    f = pdx.lib().pd_head_blocks
    f.restype, f.argtypes = ctypes.c_int64, [ctypes.c_int64, ctypes.c_int32, ctypes.c_int32]
    for c_in in (64, 128):
        for fp8 in (0, 1):
            for voxels in (1, 1000, 1 << 20, 1 << 28, (1 << 31) - 1):
                assert 1 <= f(voxels, c_in, fp8) <= (2 ** 32 - 1) // 256
            lanes = c_in // (16 if fp8 else 8)
            assert f(1000, c_in, fp8) == -(-1000 * lanes // 256)


# Networks and sizes whose launches reach the small-launch kernel's instances
REACH_NETS = [(a, network(a, w, k), None, ("bf16",) if k == 5 else ("bf16", "fp8")) for a, w, k in [
    ("plaquette", [64, 64, 64], 3), ("plaquette", [128, 128, 64], 3), ("plaquette", [64, 128, 128], 3),
    ("paper", [256, 256, 64], 3), ("paper", [64, 256], 3), ("paper", [64, 64], 5), ("paper", [128, 128], 5)]]
REACH_NETS += [("paper", None, workload.resnet_blocks([w, w]), ("bf16", "fp8")) for w in (64, 128, 256, 512)]
REACH_NETS += [("paper", None, [(4, a, a, 1), (a, b, b, 1), (b, b, 4, 1)], ("bf16",)) for a, b in ((64, 128), (128, 64))]
REACH_SIZES = [(d, T, b) for d in (3, 5, 9, 11, 13, 21, 31, 43) for T in sorted({1, 2, 3, 5, d})
               for b in (1, 2, 3, 4, 6, 8, 11, 16, 24, 36, 48, 72, 100, 150, 250, 400)
               if b == 1 or b * T * d * d < 150000]


def test_every_small_launch_instance_is_tested():
    """What the networks and sizes above reach is run by the GPU tests' cases."""
    pytest.importorskip("torch")
    import test_gpu_small_launch as cases
    from resnet_cases import RESNET_CASES, RESNET_FP8_CASES
    tested = set()
    for layout, widths, k, d, T, batch, dtype in cases.CASES:
        tested |= small_instances(d, T, dtype, batch, network(layout, widths, k), None, layout)
    for c in RESNET_CASES + cases.SHORTCUT_CASES + [dict(c, dtype="fp8") for c in RESNET_FP8_CASES]:
        tested |= small_instances(c["d"], c["T"], c.get("dtype", "bf16"), c["B"], None, c["blocks"], c["layout"])
    reached = set()
    for layout, layers, blocks, dtypes in REACH_NETS:
        for dtype in dtypes:
            for d, T, batch in REACH_SIZES:
                reached |= small_instances(d, T, dtype, batch, layers, blocks, layout)
    assert len(reached) > 80 and reached <= tested, sorted(reached - tested)


def test_the_fp32_tests_run_every_kind_of_tile():
    """Tiles of 16 to 64 voxels by 16 to 128 channels: layer 1, chunks of 8 and 16 channels, the head."""
    pytest.importorskip("torch")
    import test_gpu_fp32 as cases

    def tiles(widths, d, T, batch):
        layers = network("plaquette", widths)
        for r in launches(d, T, "fp32", batch, layers):
            ci = layers[r.layer][0]
            yield ("first" if ci == 2 else "c8" if ci % 16 else "c16", r.layer == len(widths) - 1, r.rows, r.cols)

    tested = {t for c in cases.CASES + cases.TILES for t in tiles(*c)}
    reached = {t for w in ([8] * 2, [24] * 3, [32] * 4, [64] * 6, [40, 56, 64], [72, 104, 120], [96, 112, 128], [128] * 2,
                           [16, 48, 80], [64], [128], [24], [48], [80])
               for d in (3, 5, 9, 13) for batch in (1, 4, 16, 32, 64, 128, 200, 300) for t in tiles(w, d, d, batch)
               if batch * d * (d + 1) ** 2 < 200000}
    assert reached <= tested, sorted(reached - tested)
