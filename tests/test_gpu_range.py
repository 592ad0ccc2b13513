"""Amplitudes at both ends of float32 on the line-pair kernels (whole-array registers, bands, long axes): a
single value of 3e38 and amplitudes of FLT_MAX / sqrt(rows cols), whose exact transforms are
representable, stay finite and meet the usual gates; subnormal arrays keep their bits.

The subnormal bound: U[-1, 1] * 1e-40 has an rms of 41,000 spacings (2^-149), so 8e-5 allows an rms
error of 3.3 spacings, the noise of 130 independent roundings per value; a separable transform rounds
its subnormal results about a dozen times."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import GATE, reference

pytestmark = pytest.mark.gpu
FLT_MAX = float(np.finfo(np.float32).max)
SHAPES = [(256, 256), (128, 256), (256, 128), (64, 256), (256, 64), (32, 128), (128, 64), (8, 128), (16, 256), (128, 8),
          (256, 16), (512, 512), (1024, 256), (8, 1024), (1024, 8), (512, 64)]


def _run(x, direction):
    import torch
    import paper_2609_28519_amd as dct
    dct.init(0)
    h, w = x.shape[1:]
    if max(h, w) <= 256:  # the variant of large batches, whatever this one's size
        dct.set_variant(h, w, direction, "fp32", dct.get_variant(h, w, direction, "fp32"))
    y = dct.transform(torch.from_numpy(x).cuda(), None, direction, "fp32")
    return y.cpu().numpy()


def _scored(x, direction):
    """The largest e_rel, with inputs and outputs scaled by 2^-40 first so that norms stay finite."""
    y = _run(x, direction)
    assert np.isfinite(y).all(), (x.shape, direction, np.isfinite(y).mean())
    s = 2.0 ** -40
    xs = x.astype(np.float64) * s
    ref = {"forward": oracle.forward, "inverse": oracle.inverse}.get(direction, lambda v: v)(xs)
    return oracle.e_rel(y.astype(np.float64) * s, ref, xs).max()


@pytest.mark.parametrize("h,w", SHAPES)
def test_single_large_value(h, w):
    g = np.random.default_rng(h * 31 + w)
    x = np.zeros((4, h, w), np.float32)
    x.reshape(4, -1)[np.arange(4), g.integers(0, h * w, 4)] = 3e38
    for d in ("forward", "inverse"):
        e = _scored(x, d)
        assert e <= GATE[d], (h, w, d, e)


@pytest.mark.parametrize("h,w", SHAPES)
def test_large_amplitude(h, w):
    g = np.random.default_rng(h * 37 + w)
    x = (g.uniform(-1, 1, (4, h, w)) * FLT_MAX / np.sqrt(h * w)).astype(np.float32)
    for d in GATE:
        e = _scored(x, d)
        assert e <= GATE[d], (h, w, d, e)


@pytest.mark.parametrize("h,w", SHAPES)
def test_subnormal_arrays(h, w):
    g = np.random.default_rng(h * 41 + w)
    x = (g.uniform(-1, 1, (4, h, w)) * 1e-40).astype(np.float32)
    for d in GATE:
        e = oracle.e_rel(_run(x, d), reference(x, d), x).max()
        assert e <= 8e-5, (h, w, d, e)
