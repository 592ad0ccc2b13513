"""GPU parity of the band kernels (one axis 8 or 16, the other 128 or 256): every shape and direction,
batches that fill no tile, a whole one, whole workgroups and a part of the last, against the FP64 oracle;
the filter with multipliers of one reproduces the round trip bit for bit and follows the oracle otherwise."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import GATE, reference

pytestmark = pytest.mark.gpu
SHAPES = [s for a in (8, 16) for b in (128, 256) for s in ((a, b), (b, a))]


@pytest.mark.parametrize("h,w", SHAPES)
def test_band(h, w):
    import torch
    import paper_2609_28519_amd as dct
    dct.init(0)
    dirs = ("forward", "inverse", "roundtrip", "filter")
    keep = {d: dct.get_variant(h, w, d, "fp32") for d in dirs}
    tile = 4096 // (h * w)
    v = dct.variant_count(h, w, "forward", "fp32") - 1
    try:
        for d in dirs:
            dct.set_variant(h, w, d, "fp32", v)
        for batch in (1, tile, 4 * tile, 5 * tile + 1):
            g = np.random.default_rng(h * 100 + w + batch)
            x = g.standard_normal((batch, h, w)).astype(np.float32)
            x[0] *= np.float32(2.0) ** 60
            t = torch.from_numpy(x).cuda()
            for d in dirs[:3]:
                y = dct.transform(t, None, d, "fp32")
                e = oracle.e_rel(y.cpu().numpy(), reference(x, d), x)
                assert e.max() <= GATE[d], (h, w, v, batch, d, e.max())
                z = t.clone()
                dct.transform(z, z, d, "fp32")
                assert torch.equal(z, y), (h, w, v, batch, d)
            assert torch.equal(dct.filter(t, torch.ones(h, w, device="cuda")), y), (h, w, v, batch)
            lam = g.uniform(-2, 2, x.shape).astype(np.float32)
            f = dct.filter(t, torch.from_numpy(lam).cuda()).cpu().numpy()
            off = np.sqrt(((f - oracle.filter(x, lam.astype(np.float64))) ** 2).sum(axis=(1, 2)))
            scale = np.abs(lam).max(axis=(1, 2)) * np.sqrt((x.astype(np.float64) ** 2).sum(axis=(1, 2)))
            assert (off / scale).max() <= GATE["roundtrip"], (h, w, v, batch)
    finally:
        for d, k in keep.items():
            dct.set_variant(h, w, d, "fp32", k)
