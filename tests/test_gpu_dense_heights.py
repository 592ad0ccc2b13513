"""Image heights that take the dense product (a prime factor so large that mix_plan leaves the length out: 131,
262, 997, 1021): through the workspace of ragged plans (several classes, images and heights), in place, and
through dct2d_image_transform_noalloc's fixed scratch in more than one chunk and on what an earlier call left
there."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import GATE, reference
from tests.test_gpu_ragged_families import run_plan

pytestmark = pytest.mark.gpu
DIRS = ("forward", "inverse", "roundtrip")


# recorded as a chain of classes, and as a fork (more classes; more floats)
SMALL = {(131, 24): 3, (262, 12): 4, (8, 8): 9}
MANY = {**SMALL, (131, 40): 2, (997, 12): 5, (40, 24): 2, (64, 64): 5, (64, 100): 3}
LARGE = {**SMALL, (1024, 1024): 9}


@pytest.mark.parametrize("direction", DIRS)
@pytest.mark.parametrize("counts", (SMALL, MANY, LARGE), ids=("small", "many", "large"))
def test_ragged_dense_heights(direction, counts):
    for _ in run_plan(counts, direction, 31):
        pass


@pytest.mark.parametrize("direction", DIRS)
def test_noalloc_chunks_and_leftovers(direction):
    import torch
    import paper_2609_28519_amd as dct
    dct.init(0)
    # 15 images of 1021 x 1024 fill the 64 MiB beside their table, 1999 of 131 x 64; the calls in between find
    # a larger call's table and workspace in the scratch
    for h, w, batch, look in ((1021, 1024, 20, (0, 14, 15, 19)), (997, 600, 3, (0, 2)), (131, 64, 2100, (0, 1998, 1999, 2099))):
        x = np.random.default_rng(h + w).uniform(-1, 1, (batch, h, w)).astype(np.float32)
        t = torch.from_numpy(x).cuda()
        ref = dct.image_transform(t, None, direction)
        got = dct.image_transform(t, torch.full_like(t, float("nan")), direction, noalloc=True)
        assert torch.equal(ref, got), (h, w, direction)
        assert torch.equal(t, torch.from_numpy(x).cuda()), (h, w, direction)
        for noalloc in (False, True):
            z = t.clone()
            assert torch.equal(dct.image_transform(z, z, direction, noalloc=noalloc), ref), (h, w, direction, noalloc)
        pick = list(look)
        e = oracle.e_rel(got[pick].cpu().numpy(), reference(x[pick], direction), x[pick])
        assert e.max() <= GATE[direction], (h, w, direction, e.max())
