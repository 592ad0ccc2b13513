"""The rules that choose kernels on the host, called in the built library without a GPU: which variant a
ragged plan runs where the policy names another, and which plans record their classes as a chain."""
import ctypes

import pytest

import paper_2609_28519_amd as dct

SHAPES = [(a, b) for a in (8, 16, 32, 64, 128, 256) for b in (8, 16, 32, 64, 128, 256)]
# k_rect256_db loops over the batch with one workgroup per CU; its one-array-per-workgroup form is k_rect256
LOOPING = {(256, 64, 1): (3, 0), (256, 32, 1): (3, 0)}


def _rule(name, *args):
    fn = getattr(dct.load(), "_ZN3dct%d%sE%s" % (len(name), name, "i" * len(args)))
    fn.restype = ctypes.c_int
    return fn(*(ctypes.c_int(a) for a in args))


@pytest.mark.parametrize("h,w", SHAPES)
def test_ragged_plans_keep_the_kernel_of_every_default(h, w):
    first = 1 << 30 if max(h, w) <= 64 else _rule("fp32_tile_variant", h, w)  # the first of k_tile / k_band
    for d in range(3):
        v = _rule("fp32_default_variant", h, w, d)
        u = _rule("fp32_unshared_variant", h, w, v)
        assert 0 <= u < _rule("fp32_variant_count", h, w, d), (h, w, d, v, u)
        if (h, w, d) in LOOPING:
            assert (v, u) == LOOPING[h, w, d]
        else:
            assert u == (first if v >= first else v), (h, w, d, v, u)


@pytest.mark.parametrize("h,w", SHAPES)
def test_every_late_variant_maps_to_its_one_array_form(h, w):
    if max(h, w) <= 64:
        return
    first = _rule("fp32_tile_variant", h, w)
    for v in range(first, _rule("fp32_variant_count", h, w, 0)):
        assert _rule("fp32_unshared_variant", h, w, v) == first, (h, w, v)


def test_plans_of_many_classes_are_not_chained():
    """A chain takes 7 us per kernel, so only few classes and little data make one."""
    fn = dct.load()._ZN3dct16records_as_chainEli
    fn.restype = ctypes.c_bool
    chain = lambda floats, nodes: fn(ctypes.c_int64(floats), ctypes.c_int(nodes))  # noqa: E731
    assert chain(1 << 20, 1) and chain(1 << 23, 8)
    assert not chain((1 << 23) + 1, 8) and not chain(1 << 20, 9) and not chain(1 << 18, 36)
