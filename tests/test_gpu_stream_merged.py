"""GPU: a stream's windows of all lengths and boundary kinds run as one batch.

The first and last windows read further rounds instead of being shorter, and
the geometric channels are cleared for their samples only, so every
combination of bases is compared with the GPU's own run over the whole stream
(sites whose logit is within the bf16 bound excused), on streams of a few
windows, of one window's length or less, with a ragged last core, and with a
buffer of exactly the receptive field."""
import numpy as np
import pytest

import oracle
import paper_2604_12841_amd as pdx
from paper_2604_12841_amd import workload
from launch_plan import stream_batches
from parity import assert_parity, compare, dev_u64, host_u64, run_gpu, say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cuda():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda")


@pytest.mark.parametrize("d,n,core,buffer,B,first,last,dtype", [
    (13, 100, 13, 13, 4, "Z", "X", "bf16"),
    (13, 90, 13, 13, 4, "X", None, "bf16"),
    (13, 77, 20, 3, 5, None, "Z", "bf16"),
    (13, 30, 13, 13, 6, "X", "Z", "bf16"),
    (11, 64, 11, 11, 3, "Z", "Z", "fp8"),
], ids=lambda v: str(v))
def test_windows_in_one_batch(cuda, d, n, core, buffer, B, first, last, dtype):
    layers = workload.paper_layer_spec([64, 64, 4], [3, 3, 3])
    weights = workload.he_normal_weights(layers, 401)
    det, _ = workload.make_inputs(d, n, B, 0.02, 0.02, 402)
    say("stream", d, n, core, buffer, B, first, last, dtype)
    assert stream_batches(layers, d, n, core, buffer, dtype, B) == 1
    assert stream_batches(layers, d, n, core, buffer, dtype, B, n_cu=0) > 1
    s = pdx.Stream(weights, d, n, layers, core, buffer, dtype, n_streams=B, layout="paper", first=first, last=last)
    flips = torch.full((B, s.flip_words), -1, dtype=torch.int64, device="cuda")
    res = torch.full((B, s.det_words), -1, dtype=torch.int64, device="cuda")
    s.run(dev_u64(det), flips, res)
    torch.cuda.synchronize()
    s.close()
    pre = pdx.Predecoder(weights, d, n, layers, dtype, max_batch=B, layout="paper", first=first, last=last)
    f1, r1, l1 = run_gpu(pre, det)
    pre.close()
    from parity import TOL
    st = compare(d, n, "bf16", l1.astype(np.float64), f1, r1, host_u64(flips), host_u64(res), layout="paper",
                 tol=TOL[dtype])
    say("  against the whole-stream run", st)
    if dtype == "bf16":
        assert_parity(st, "bf16")
    assert st["flip_mismatch"] == 0 and st["res_mismatch"] == 0
    np.testing.assert_array_equal(host_u64(res), oracle.residual_from_flips(d, n, det, host_u64(flips)))
