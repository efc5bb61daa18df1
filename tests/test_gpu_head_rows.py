"""GPU: the 1x1x1 head's kernel over more rows than its grid takes at once.

A one-hidden-layer network on the paper's layout; the first and the last
samples of a large batch equal the same samples run by themselves, bit by bit
(a row's sums do not depend on the batch)."""
import ctypes

import numpy as np
import pytest

import paper_2604_12841_amd as pdx
from launch_plan import network
from paper_2604_12841_amd import workload
from parity import run_gpu, say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width,B", [(128, 500), (64, 1000), (128, 3)])
def test_head_over_many_rows(width, B):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    d = T = 13
    layers = network("paper", [width])[:-1] + [(width, 4, 1, workload.NONE)]
    weights = workload.he_normal_weights(layers, 11)
    det, _ = workload.make_inputs(d, T, min(B, 50), 0.02, 0.02, 12)
    det = np.tile(det, (-(-B // len(det)), 1))[:B]
    det[-1] ^= det[0]
    say("head rows", width, B)
    f = pdx.lib().pd_head_blocks
    f.restype, f.argtypes = ctypes.c_int64, [ctypes.c_int64, ctypes.c_int32, ctypes.c_int32]
    rows = B * T * d * d
    assert (f(rows, width, 0) * 256 < rows * width // 8) == (B > 3)  # the grid takes turns
    pick = sorted({0, 1, B - 2, B - 1})
    pre = pdx.Predecoder(weights, d, T, layers, "bf16", max_batch=B, layout="paper", first="Z", last="Z")
    flips, res, logits = run_gpu(pre, det)
    pre.close()
    one = pdx.Predecoder(weights, d, T, layers, "bf16", max_batch=len(pick), layout="paper", first="Z", last="Z")
    f1, r1, l1 = run_gpu(one, det[pick])
    one.close()
    assert np.array_equal(logits[pick].view(np.int32), l1.view(np.int32))
    assert np.array_equal(flips[pick], f1) and np.array_equal(res[pick], r1)
    assert np.isfinite(logits).all()
