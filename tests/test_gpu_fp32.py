"""GPU parity of the fp32 path: the matrix-core conv over its tile shapes.

Widths with and without a remainder of 8 channels, channel blocks in one or
several groups, one hidden layer (layer 1 carries the head) and several, and
batches from one wave's worth of voxels to launches of the largest tiles,
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


@pytest.mark.parametrize("widths,d,T,B", [
    ([8], 3, 1, 1),                    # layer 1 with the head, one partial wave
    ([128], 5, 4, 3),
    ([8, 8], 3, 2, 1),                 # chunks of 8 channels only
    ([16, 24, 40], 5, 3, 2),           # remainders after full chunks, padded channel blocks
    ([32, 32, 32, 32], 5, 5, 64),      # the fp32 workload
    ([48, 72, 88], 5, 5, 7),           # blocks of 3 and more than one group
    ([96, 112, 128], 7, 3, 5),         # heads over 6, 7 and 8 blocks
    ([128, 104], 5, 3, 4),
    ([64, 56, 64], 9, 9, 100),         # the largest tiles (4 x 4 blocks)
    ([128, 128], 9, 9, 60),            # ... and 2 x 8 with the head
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, list) else str(v))
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
