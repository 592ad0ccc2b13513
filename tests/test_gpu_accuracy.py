"""Errors of the line-pair kernels, averaged over arrays of normal values: no more than a few per cent over
those of the one-line transforms of the same lengths (even/odd recursion, dct1d.hpp), which set the
library's accuracy at every other size.  The bounds are the averages measured with those on the same
shapes, times 1.08 for the forward transform and 1.05 for the round trip (two runs with other arrays differ by
less than 0.005 of that)."""
import numpy as np
import pytest

from tests.gpu_util import per_array_rel

pytestmark = pytest.mark.gpu
# shape: forward, round trip, in units of 1e-7
RECURSION = {(256, 256): (1.454, 2.196), (128, 256): (1.391, 2.117), (64, 256): (1.346, 2.007), (32, 128): (1.219, 1.814),
             (128, 64): (1.265, 1.865), (512, 512): (1.514, 2.247), (1024, 1024): (1.633, 2.422), (1024, 256): (1.545, 2.307),
             (8, 1024): (1.324, 1.992), (16, 256): (1.247, 1.883)}


def _q(n):
    import torch
    k, j = np.arange(n)[:, None], np.arange(n)[None, :]
    q = np.cos(np.pi * ((k * (2 * j + 1)) % (4 * n)) / (2 * n)) * np.sqrt(2.0 / n)
    q[0] = np.sqrt(1.0 / n)
    return torch.from_numpy(q).cuda()


@pytest.mark.parametrize("h,w", sorted(RECURSION))
def test_mean_error(h, w):
    import torch
    import paper_2609_28519_amd as dct
    dct.init(0)
    g = torch.Generator(device="cuda")
    g.manual_seed(h * 1031 + w)
    b = max(4, (1 << 22) // (h * w))
    x = torch.randn(b, h, w, generator=g, device="cuda")
    rows = x.double().reshape(b * h, w) @ _q(w).t().contiguous()
    cols = rows.reshape(b, h, w).transpose(1, 2).reshape(b * w, h) @ _q(h).t().contiguous()
    exact = cols.reshape(b, w, h).transpose(1, 2).contiguous()
    forward, roundtrip = RECURSION[h, w]
    e = per_array_rel(dct.transform(x, None, "forward", "fp32"), exact).mean()
    assert e <= 1.08e-7 * forward, (h, w, "forward", e)
    e = per_array_rel(dct.transform(x, None, "roundtrip", "fp32"), x).mean()
    assert e <= 1.05e-7 * roundtrip, (h, w, "roundtrip", e)
