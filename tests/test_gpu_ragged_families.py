"""Ragged plans over the kernel families of rectangles, which they reach through offset lists and the plan's
base slot: every k_tile, k_band and k_pack shape with a few arrays each, in mixed order with gaps, and
k_pack on padded strides of the basic calls.  A plan runs the kernel that the policy names (or its
one-array-per-workgroup form), so its results are those of the basic call bit for bit."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import GATE, reference

pytestmark = pytest.mark.gpu
DIRS = ("forward", "inverse", "roundtrip")
P = (8, 16, 32, 64, 128, 256)
RECTS = [(a, b) for a in P for b in P if a != b] + [(256, 256)]
GUARD = np.float32(-7.25)
# their inverse loops over the batch (k_rect256_db); a plan runs k_rect256
OTHER_KERNEL = {(256, 64, "inverse"), (256, 32, "inverse")}


def layout(counts, seed, gap=16):
    """{shape: count} -> offsets, rows, cols in mixed order with guard gaps, and the buffer's size."""
    items = [s for s, k in counts.items() for _ in range(k)]
    items = [items[i] for i in np.random.default_rng(seed).permutation(len(items))]
    rows, cols = (np.array(v, np.int32) for v in zip(*items))
    offsets = gap + np.concatenate([[0], np.cumsum(rows.astype(np.int64) * cols + gap)])
    return offsets[:-1], rows, cols, int(offsets[-1])


def run_plan(counts, direction, seed):
    """Executes a plan twice (two buffers) and checks guards, replay and every item against the oracle;
    yields (shape, inputs, outputs)."""
    import torch
    import paper_2609_28519_amd as dct
    dct.init(0)
    offsets, rows, cols, size = layout(counts, seed)
    data = np.full(size, GUARD, np.float32)
    g = np.random.default_rng(seed + 1)
    inside = np.zeros(size, bool)
    for o, h, w in zip(offsets, rows, cols):
        data[o:o + h * w] = g.standard_normal(int(h) * int(w))
        inside[o:o + h * w] = True
    plan = dct.RaggedPlan(offsets, rows, cols, direction, "fp32")
    assert plan.info()["classes"] == len(counts)
    bufs = [torch.from_numpy(data).cuda() for _ in range(2)]
    for b in bufs:
        plan.execute(b)
    torch.cuda.synchronize()
    out = bufs[0].cpu().numpy()
    assert np.array_equal(out, bufs[1].cpu().numpy())
    assert (out[~inside] == GUARD).all()
    plan.close()
    for h, w in counts:
        at = [int(o) for o, r, c in zip(offsets, rows, cols) if (r, c) == (h, w)]
        x, y = (np.stack([v[o:o + h * w].reshape(h, w) for o in at]) for v in (data, out))
        e = oracle.e_rel(y, reference(x, direction), x)
        assert e.max() <= GATE[direction], (h, w, direction, e.max())
        yield (h, w), x, y


@pytest.mark.parametrize("direction", DIRS)
def test_rectangles(direction):
    import torch
    import paper_2609_28519_amd as dct
    counts = {s: 1 + 2 * (i % 4) + 60 * (max(s) <= 32) for i, s in enumerate(RECTS)}
    for (h, w), x, y in run_plan(counts, direction, 5):
        if (h, w, direction) not in OTHER_KERNEL:
            z = dct.transform(torch.from_numpy(x).cuda(), None, direction, "fp32").cpu().numpy()
            assert np.array_equal(z, y), (h, w, direction)


@pytest.mark.parametrize("h,w", [s for s in RECTS if max(s) <= 64])
@pytest.mark.parametrize("pad", (4, 20))
def test_pack_padded_strides(h, w, pad):
    import torch
    import paper_2609_28519_amd as dct
    dct.init(0)
    n, stride = 64 // min(h, w) + 3, h * w + pad
    x = np.random.default_rng(h * 100 + w).standard_normal((n, h, w)).astype(np.float32)
    names = {"forward": dct.forward_, "inverse": dct.inverse_, "roundtrip": dct.roundtrip_}
    keep = {d: dct.get_variant(h, w, d, "fp32") for d in DIRS}
    try:
        for d in DIRS:
            dct.set_variant(h, w, d, "fp32", 13)
            buf = torch.full((n * stride,), float(GUARD), device="cuda")
            buf.view(n, stride)[:, :h * w] = torch.from_numpy(x).cuda().view(n, -1)
            names[d](buf, h, w, stride)
            y = dct.transform(torch.from_numpy(x).cuda(), None, d, "fp32")
            assert torch.equal(buf.view(n, stride)[:, :h * w].reshape(n, h, w), y), (h, w, d)
            assert (buf.view(n, stride)[:, h * w:] == float(GUARD)).all(), (h, w, d)
            e = oracle.e_rel(y.cpu().numpy(), reference(x, d), x)
            assert e.max() <= GATE[d], (h, w, d, e.max())
    finally:
        for d, k in keep.items():
            dct.set_variant(h, w, d, "fp32", k)
