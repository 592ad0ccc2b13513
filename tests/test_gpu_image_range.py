"""Large amplitudes on whole images: as with a product with Q_n, whose intermediate values are no larger than
its result can be, constant images, random ones and single values stay finite up to a small factor
below what the result can represent, and meet the usual gates.  Both kinds of axis: mixed-radix lengths, powers
of two by line pairs (256 and more) and by one thread per line (below)."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import GATE

pytestmark = pytest.mark.gpu
FLT_MAX = float(np.finfo(np.float32).max)
SHAPES = [(512, 384), (384, 512), (600, 1000), (24, 40), (13, 52), (255, 256), (1000, 12), (822, 12), (137, 712), (257, 384),
          (100, 64), (64, 100), (24, 128), (128, 24), (12, 8), (8, 12), (1024, 20), (20, 1024), (997, 64)]


def _scored(x, direction):
    """The largest e_rel, with inputs and outputs scaled by 2^-40 first so that norms stay finite."""
    import torch
    import paper_2609_28519_amd as dct
    dct.init(0)
    y = dct.image_transform(torch.from_numpy(x).cuda(), None, direction).cpu().numpy()
    assert np.isfinite(y).all(), (x.shape, direction, np.isfinite(y).mean())
    s = 2.0 ** -40
    xs = x.astype(np.float64) * s
    ref = {"forward": oracle.forward, "inverse": oracle.inverse}.get(direction, lambda v: v)(xs)
    e = oracle.e_rel(y.astype(np.float64) * s, ref, xs).max()
    assert e <= GATE[direction], (x.shape, direction, e)


def test_constant_image_with_a_representable_sum():
    _scored(np.full((1, 512, 384), 5e35, np.float32), "forward")  # largest coefficient 2.2e38


@pytest.mark.parametrize("h,w", SHAPES)
def test_single_large_value(h, w):
    g = np.random.default_rng(h * 31 + w)
    x = np.zeros((4, h, w), np.float32)
    x.reshape(4, -1)[np.arange(4), g.integers(0, h * w, 4)] = 3e38
    for d in ("forward", "inverse"):
        _scored(x, d)


@pytest.mark.parametrize("h,w", SHAPES)
def test_large_amplitude(h, w):
    g = np.random.default_rng(h * 37 + w)
    top = FLT_MAX / np.sqrt(h * w)  # the sum of a constant image of this value is FLT_MAX
    random = g.uniform(-1, 1, (1, h, w)) * top
    mode = np.cos(np.pi * (np.arange(h)[:, None] + 0.5) * (h // 3) / h) * np.cos(np.pi * (np.arange(w) + 0.5) * (w // 5) / w)
    x = np.concatenate([random, np.full((1, h, w), top / 4), (mode * top / 4)[None]]).astype(np.float32)
    for d in GATE:
        _scored(x, d)
