"""GPU parity of the fp32 path: the matrix-core conv over its tile shapes.

Widths with and without a remainder of 8 channels, channel blocks in one or
several groups, one hidden layer (layer 1 carries the head) and several, and
batches from one wave's worth of voxels to launches of the largest tiles
(tests/test_launch_plan.py checks that every tile the choice takes is run),
against the CPU oracle under the fp32 parity rule (logits within 1e-4, which
is above the bound of an fp32 chain of 27 x 128 terms of these magnitudes)."""
import numpy as np
import pytest

import oracle
import paper_2604_12841_amd as pdx
from paper_2604_12841_amd import workload
from parity import assert_parity, compare, dev_u64, host_u64, run_gpu, say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cuda():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda")


CASES = [
    ([8], 3, 1, 1),                    # layer 1 with the head, one partial wave
    ([128], 5, 4, 3),
    ([8, 8], 3, 2, 1),                 # chunks of 8 channels only
    ([16, 24, 40], 5, 3, 2),           # remainders after full chunks, padded channel blocks
    ([32, 32, 32, 32], 5, 5, 64),      # the fp32 workload
    ([48, 72, 88], 5, 5, 7),           # blocks of 3 and more than one group
    ([96, 112, 128], 7, 3, 5),         # heads over 6, 7 and 8 blocks
    ([128, 104], 5, 3, 4),
    ([64, 56, 64], 9, 9, 100),         # 2 x 4 blocks
    ([128, 128], 9, 9, 60),            # 2 x 8 with the head
    ([64, 64, 64], 9, 9, 128),         # the largest tiles, 4 x 4 blocks
    ([64, 64, 64], 9, 9, 127),         # ... with a last wave that is not full
    ([56, 64, 8], 9, 9, 128),          # ... over chunks of 8 channels
]

# The other tiles of 1, 2 and 4 x 16 voxels by 1 to 8 x 16 channels, the smallest networks and batches that run them
TILES = [
    ([24, 40, 56], 3, 1, 1), ([24], 3, 1, 1), ([40], 3, 1, 1), ([56], 3, 1, 1), ([72], 3, 1, 1), ([16, 8], 3, 1, 1),
    ([88], 3, 1, 1), ([104], 3, 1, 1), ([8, 24], 3, 1, 1), ([8, 72], 3, 1, 1), ([16, 40], 3, 1, 1), ([8, 104], 3, 1, 1),
    ([16, 56], 3, 1, 1), ([8, 120], 3, 1, 1), ([16, 72], 3, 1, 1), ([16, 88], 3, 1, 1), ([16, 48, 80], 7, 2, 130),
    ([24, 40, 56], 9, 5, 100), ([104, 8], 7, 2, 130), ([24, 40, 56], 7, 2, 130), ([104, 8], 3, 2, 130),
    ([8, 8], 9, 5, 100), ([24, 40, 56], 7, 1, 100), ([104, 8], 7, 1, 130), ([24, 40, 56], 7, 1, 130),
    ([16, 48, 80], 7, 1, 130), ([8], 7, 2, 130), ([24], 7, 2, 130), ([40], 7, 2, 130), ([56], 7, 2, 130),
    ([72], 7, 2, 130), ([16, 8], 7, 2, 130), ([88], 7, 2, 130), ([104], 7, 2, 130), ([8, 24], 7, 2, 130),
    ([120], 7, 2, 130), ([8, 40], 7, 2, 130), ([16, 24], 7, 2, 130), ([8, 72], 7, 2, 130), ([16, 40], 7, 2, 130),
    ([8, 88], 7, 2, 130), ([8, 104], 7, 2, 130), ([16, 56], 7, 2, 130), ([8, 120], 7, 2, 130), ([16, 88], 7, 2, 130),
    ([16, 104], 7, 2, 130), ([104, 8], 9, 2, 130), ([24], 9, 9, 40), ([8, 24], 9, 9, 40), ([16, 24], 7, 9, 64),
    ([8], 9, 5, 100), ([40], 9, 5, 100), ([56], 9, 5, 100), ([16, 8], 9, 5, 100), ([8, 40], 9, 5, 100),
    ([16, 40], 9, 5, 100), ([16, 56], 9, 5, 100), ([16, 48, 80], 9, 5, 100), ([8, 104, 8], 7, 1, 100),
    ([8, 72, 8], 7, 1, 130), ([16, 72, 8], 7, 1, 130), ([8, 104, 8], 3, 5, 150), ([8, 8, 8], 7, 2, 130),
    ([16, 8, 8], 7, 2, 130), ([8, 72, 8], 7, 2, 130), ([16, 72, 8], 7, 2, 130), ([8, 104, 8], 9, 2, 128),
    ([8, 8, 8], 9, 5, 100), ([16, 8, 8], 9, 5, 100),
]


@pytest.mark.parametrize("widths,d,T,B", CASES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, list) else str(v))
@pytest.mark.parametrize("act", ["gelu", "relu"])
def test_fp32_network(cuda, widths, d, T, B, act):
    a = {"gelu": workload.GELU_TANH, "relu": workload.RELU}[act]
    layers, ci = [], 2
    for w in widths:
        layers.append((ci, w, 3, a))
        ci = w
    layers.append((ci, 4, 1, workload.NONE))
    weights = workload.he_normal_weights(layers, seed=5 + len(widths) + widths[0])
    det, _ = workload.make_inputs(d, T, B, 0.02, 0.02, seed=9)
    pre = pdx.Predecoder(weights, d, T, layers, "fp32", max_batch=B)
    say("fp32 network", widths, "d", d, "T", T, "B", B, act)
    flips, res, logits = run_gpu(pre, det)
    n = min(B, 4)  # the oracle on the first and last samples
    pick = np.r_[0:(n + 1) // 2, B - n // 2:B]
    ref = oracle.run(d, T, det[pick], layers, weights, bf16=False)
    st = compare(d, T, "fp32", *ref, flips[pick], res[pick], logits[pick])
    assert_parity(st, "fp32")
    assert np.isfinite(logits).all()
    # without logits, the same bits
    f2 = torch.full((B, pre.flip_words), -1, dtype=torch.int64, device="cuda")
    r2 = torch.full((B, pre.det_words), -1, dtype=torch.int64, device="cuda")
    pre.run(dev_u64(det), f2, r2)
    torch.cuda.synchronize()
    assert np.array_equal(host_u64(f2), flips) and np.array_equal(host_u64(r2), res)
    pre.close()


@pytest.mark.parametrize("widths,d,T,B", TILES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, list) else str(v))
def test_fp32_tiles(cuda, widths, d, T, B):
    test_fp32_network(cuda, widths, d, T, B, "gelu")
