"""Batches of narrow images beyond what one launch holds (2^32 threads, 2^31 line pairs): computed in
parts, like any other batch."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import GATE, reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,w,batch", [(9, 8, 430_000_001), (36, 36, 31_000_001), (8, 12, 365_000_001)])
def test_more_than_one_launch_holds(h, w, batch):
    import torch
    import paper_2609_28519_amd as dct
    dct.init(0)
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < batch * h * w * 4 + (4 << 30):
        pytest.skip("not enough device memory")
    x = torch.zeros(batch, h, w, device="cuda")
    try:
        per = (1 << 34) // (h * w)
        at = sorted({0, 1, batch // 2, batch - 2, batch - 1} | {min(batch - 1, k * per + d) for k in (1, 2) for d in (-1, 0)})
        vals = np.random.default_rng(h).standard_normal((len(at), h, w)).astype(np.float32)
        for noalloc in (False, True):
            for i, v in zip(at, vals):
                x[i] = torch.from_numpy(v).cuda()
            for d in ("forward", "inverse"):
                before = x[at].cpu().numpy()
                dct.image_transform(x, x, d, noalloc=noalloc)
                e = oracle.e_rel(x[at].cpu().numpy(), reference(before, d), before)
                assert e.max() <= GATE[d], (h, w, d, noalloc, e.max())
        x[at] = 0
        assert not torch.stack([part.any() for part in torch.split(x, 1 << 24)]).any()  # nothing else was written
    finally:
        del x
        torch.cuda.empty_cache()
