"""GPU parity of k_tile (both axes 32 .. 256, one of 128 or 256): every shape, direction and both
schedules, a single array and more arrays than there are workgroups on the GPU, against the FP64
oracle at the gates used everywhere; the filter against the oracle's filter and, with multipliers of
one, bit for bit against the round trip of the same variant."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import GATE, per_array_rel, reference, spread

pytestmark = pytest.mark.gpu
SHAPES = [(256, 256), (256, 128), (128, 256), (256, 64), (64, 256), (256, 32), (32, 256), (128, 64), (64, 128),
          (128, 32), (32, 128)]
FIRST = {(256, 256): 5, (256, 128): 3, (128, 256): 3, (256, 64): 4, (64, 256): 4, (256, 32): 4, (32, 256): 4}


@pytest.mark.parametrize("h,w", SHAPES)
@pytest.mark.parametrize("more", (0, 1))
def test_tile_variants(h, w, more):
    import torch
    import paper_2609_28519_amd as dct
    dct.init(0)
    v = FIRST.get((h, w), 2) + more
    keep = {d: dct.get_variant(h, w, d, "fp32") for d in ("forward", "inverse", "roundtrip", "filter")}
    try:
        for d in keep:
            dct.set_variant(h, w, d, "fp32", v)
        # one array, and a batch past the resident workgroups of 256 CUs (1024 threads each)
        for batch in (1, 256 * 1024 // (h * w // 64) + 3):
            x = np.random.default_rng(h + w + batch).standard_normal((batch, h, w)).astype(np.float32)
            t = torch.from_numpy(x).cuda()
            at = spread(batch, 12)
            for d in ("forward", "inverse", "roundtrip"):
                y = dct.transform(t, None, d, "fp32")
                e = oracle.e_rel(y[torch.from_numpy(at).cuda()].cpu().numpy(), reference(x[at], d), x[at])
                assert e.max() <= GATE[d], (h, w, v, batch, d, e.max())
                z = t.clone()
                dct.transform(z, z, d, "fp32")
                assert torch.equal(z, y), (h, w, v, batch, d)
            assert per_array_rel(y, t).max() <= GATE["roundtrip"]
            one = dct.filter(t, torch.ones(h, w, device="cuda"))
            assert torch.equal(one, y), (h, w, v, batch)
            lam = np.random.default_rng(3).uniform(-2, 2, x[at].shape).astype(np.float32)
            f = dct.filter(torch.from_numpy(x[at]).cuda(), torch.from_numpy(lam).cuda())
            ref = oracle.filter(x[at], lam.astype(np.float64))
            off = np.sqrt(((f.cpu().numpy() - ref) ** 2).sum(axis=(1, 2)))
            scale = np.abs(lam).max(axis=(1, 2)) * np.sqrt((x[at].astype(np.float64) ** 2).sum(axis=(1, 2)))
            assert (off / scale).max() <= GATE["roundtrip"], (h, w, v, batch)
    finally:
        for d, k in keep.items():
            dct.set_variant(h, w, d, "fp32", k)
