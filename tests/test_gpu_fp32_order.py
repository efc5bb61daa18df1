"""GPU: every fp32 sum is one fma chain in a fixed order, bit by bit.

An output starts at its bias and adds weight times input over the taps and,
within a tap, the input channels in order; a logit starts at the head's bias
and runs over its channels.  So the logits, and with them the bits of sites
whose logit is near zero, do not depend on the tiles or the batch.  The chain
is recomputed here with exactly rounded fmas; ReLU networks, whose activation
rounds nothing.  Widths: chunks of 8 and 16 channels in every combination of
reading and storing, padded row blocks, one hidden layer and several, heads of
one to eight blocks."""
import numpy as np
import pytest

import paper_2604_12841_amd as pdx
from paper_2604_12841_amd import workload
from parity import run_gpu, say

torch = pytest.importorskip("torch")


def fma32(a, b, c):
    """fp32 a b + c rounded once: the product is exact in fp64, the sum is rounded to odd there."""
    p = a.astype(np.float64) * b.astype(np.float64)
    c = np.broadcast_to(c.astype(np.float64), p.shape)
    s = p + c
    t = s - p
    err = (p - (s - t)) + (c - t)
    even = (s.view(np.int64) & 1) == 0
    s = np.where((err != 0) & even, np.nextafter(s, np.where(err > 0, np.inf, -np.inf)), s)
    return s.astype(np.float32)


def test_fma32():
    one, e = np.float32(1), np.float32(2.0 ** -24)
    tiny = np.float32(2.0 ** -60)
    a = np.array([one, one, one + 2 * e, e], dtype=np.float32)
    b = np.array([e, -e, one + 2 * e, e], dtype=np.float32)
    c = np.array([one, one, tiny, one + 2 * e], dtype=np.float32)
    from fractions import Fraction
    for x, y, z, got in zip(a, b, c, fma32(a, b, c)):
        exact = Fraction(float(x)) * Fraction(float(y)) + Fraction(float(z))
        near = [got, np.nextafter(got, np.float32(-9)), np.nextafter(got, np.float32(9))]
        d = [abs(Fraction(float(v)) - exact) for v in near]
        assert d[0] <= min(d[1:])
        if d[0] in d[1:]:  # a tie goes to the even one
            assert got.view(np.int32) & 1 == 0


def chain(x, w, b):
    """x [T][H][H][ci], w [co][ci][k][k][k], b [co], all fp32; zero halo of (k - 1) / 2."""
    T, H, _, ci = x.shape
    k = w.shape[2]
    h = k // 2
    xp = np.pad(x, ((h, h), (h, h), (h, h), (0, 0)))
    y = np.broadcast_to(b, (T, H, H, b.size))
    for t in range(k):
        for i in range(k):
            for j in range(k):
                for c in range(ci):
                    y = fma32(xp[t:t + T, i:i + H, j:j + H, c, None], w[:, c, t, i, j], y)
    return y


@pytest.mark.gpu
@pytest.mark.parametrize("widths,d,T,B", [
    ([8], 3, 2, 1),
    ([40], 3, 2, 2),
    ([32, 32, 32], 3, 3, 2),
    ([8, 16, 24, 32], 3, 2, 2),
    ([24, 40, 8], 3, 2, 3),
    ([72, 48], 5, 2, 1),
    ([128, 64], 3, 2, 2),
    ([16, 128], 3, 2, 2),
    ([64, 64], 9, 9, 128),    # the largest tiles (the first and last samples are checked)
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, list) else str(v))
def test_fp32_chain(widths, d, T, B):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    layers, ci = [], 2
    for w in widths:
        layers.append((ci, w, 3, workload.RELU))
        ci = w
    layers.append((ci, 4, 1, workload.NONE))
    weights = workload.he_normal_weights(layers, seed=31 + widths[0])
    det, _ = workload.make_inputs(d, T, B, 0.05, 0.05, seed=3)
    say("fp32 chain", widths, "d", d, "T", T, "B", B)
    pre = pdx.Predecoder(weights, d, T, layers, "fp32", max_batch=B)
    _, _, logits = run_gpu(pre, det)
    planes = torch.empty((B, T, pre.grid, pre.grid, 2), dtype=torch.float32, device="cuda")
    pre.unpack(torch.from_numpy(det.view(np.int64)).cuda(), planes)
    planes = planes.cpu().numpy()
    pre.close()
    pick = sorted({0, B - 1}) if d < 9 else [B - 1]
    for s in pick:
        x, off = planes[s], 0
        if d == 9:  # the last rounds alone: two of them depend on no other
            x = x[-4:]
        for l, (ci, co, k, act) in enumerate(layers):
            n = co * ci * k ** 3
            w = weights[off:off + n].reshape(co, ci, k, k, k).astype(np.float32)
            b = weights[off + n:off + n + co].astype(np.float32)
            off += n + co
            x = chain(x, w, b)
            if act == workload.RELU:
                x = np.where(x > 0, x, np.float32(0))
        keep = 2 if d == 9 else T  # (two layers reach two rounds)
        want = x[-keep:].transpose(3, 0, 1, 2)
        got = logits[s][:, -keep:]
        assert np.array_equal(got.view(np.int32), np.ascontiguousarray(want).view(np.int32)), \
            float(np.abs(got - want).max())
