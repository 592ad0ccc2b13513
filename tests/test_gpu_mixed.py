"""GPU parity of the mixed-radix image axes: every length in [8, 1024] that is not a power of two, as
columns (any length) and as rows (multiples of 4), against the FP64 oracle at the gates used
everywhere.  Lengths with a large prime factor take the dense products, so both sides of the rule
that chooses are covered, every radix, and odd numbers of rows (a last row without a partner)."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import GATE, reference

pytestmark = pytest.mark.gpu
DIRS = ("forward", "inverse", "roundtrip")


def _check(h, w, batch, direction, noalloc=False):
    import torch
    import paper_2609_28519_amd as dct
    x = np.random.default_rng(h * 1031 + w).standard_normal((batch, h, w)).astype(np.float32)
    t = torch.from_numpy(x).cuda()
    y = dct.image_transform(t, None, direction, noalloc=noalloc)
    torch.cuda.synchronize()
    e = oracle.e_rel(y.cpu().numpy(), reference(x, direction), x)
    assert e.max() <= GATE[direction], (h, w, batch, direction, e.max())


@pytest.mark.parametrize("lo", range(8, 1025, 127))
def test_every_length(lo):
    import paper_2609_28519_amd as dct
    dct.init(0)
    for i, n in enumerate(range(lo, min(lo + 127, 1025))):
        if n & (n - 1) == 0:
            continue
        _check(n, 8, 3, DIRS[i % 3])
        if n % 4 == 0:
            _check(9, n, 2, DIRS[(i // 4) % 3])


@pytest.mark.parametrize("h,w,batch", [(601, 512, 1), (999, 1024, 1), (255, 256, 3), (12, 12, 401), (9, 8, 700),
                                       (33, 100, 67), (1000, 12, 65), (384, 512, 33), (720, 1280 // 2, 3),
                                       (1020, 1020, 1), (1021, 600, 1), (600, 1012, 2), (997, 1012, 1)])
@pytest.mark.parametrize("direction", DIRS)
def test_tiles_and_mixed_axes(h, w, batch, direction):
    _check(h, w, batch, direction)
    _check(h, w, batch, direction, noalloc=True)
