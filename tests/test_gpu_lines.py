"""GPU parity of the line-pair passes (axes of 256, 512 and 1024 in power-of-two shapes with a long
axis) where their tiling can go wrong: a single array, workgroups with missing row tiles, column
tiles of 8, 16 and 32 columns, and batches that leave a part of the last group of 128 column tiles.
Against the FP64 oracle at the gates used everywhere (2e-6 forward and inverse, 4e-6 round trip)."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import reference, run, GATE

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,w,batch", [(8, 1024, 1), (8, 1024, 7), (8, 512, 3), (512, 8, 1), (1024, 8, 129),
                                       (1024, 16, 5), (512, 16, 131), (512, 32, 33), (1024, 32, 1), (1024, 512, 5),
                                       (512, 256, 9), (256, 512, 17), (256, 1024, 2), (1024, 256, 9)])
@pytest.mark.parametrize("direction", ("forward", "inverse", "roundtrip"))
def test_line_passes_at_tile_edges(h, w, batch, direction):
    x = np.random.default_rng(h * 7 + w + batch).standard_normal((batch, h, w)).astype(np.float32)
    y = run(x, direction, "auto")
    e = oracle.e_rel(y, reference(x, direction), x)
    assert e.max() <= GATE[direction], (h, w, batch, direction, int(np.argmax(e)), e.max())
