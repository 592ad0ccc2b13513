"""The rules that choose kernels on the host, called in the built library without a GPU: which variant a
ragged plan runs where the policy names another, which plans record their classes as a chain, and which
shapes run another variant for a few arrays."""
import ctypes

import pytest

import paper_2609_28519_amd as dct

SHAPES = [(a, b) for a in (8, 16, 32, 64, 128, 256) for b in (8, 16, 32, 64, 128, 256)]
# k_rect256_db loops over the batch with one workgroup per CU; its one-array-per-workgroup form is k_rect256
LOOPING = {(256, 64, 1): (3, 0), (256, 32, 1): (3, 0)}


LARGE = 1 << 40


def _rule(name, *args):
    fn = getattr(dct.load(), "_ZN3dct%d%sE%s" % (len(name), name, "i" * len(args)))
    fn.restype = ctypes.c_int
    return fn(*(ctypes.c_int(a) for a in args))


def _default(h, w, direction, batch=LARGE):
    fn = dct.load()._ZN3dct20fp32_default_variantEiiil
    fn.restype = ctypes.c_int
    return fn(ctypes.c_int(h), ctypes.c_int(w), ctypes.c_int(direction), ctypes.c_int64(batch))


@pytest.mark.parametrize("h,w", SHAPES)
def test_ragged_plans_keep_the_kernel_of_every_default(h, w):
    first = 1 << 30 if max(h, w) <= 64 else _rule("fp32_tile_variant", h, w)  # the first of k_tile / k_band
    for d in range(3):
        v = _default(h, w, d)
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


@pytest.mark.parametrize("h,w,direction,batch,few,many", [
    (8, 64, 0, 6143, 4, 15), (64, 8, 1, 6143, 4, 15), (8, 64, 2, 4095, 4, 15), (64, 8, 3, 4095, 4, 15),
    (16, 64, 2, 4095, 4, 15), (64, 16, 3, 4095, 4, 15), (8, 128, 0, 511, 0, 2), (128, 8, 3, 511, 0, 2), (256, 64, 2, 512, 0, 4),
    (32, 64, 0, 4096, 4, 8), (64, 32, 1, 4096, 4, 8)])
def test_few_arrays_run_the_variant_that_leads_there(h, w, direction, batch, few, many):
    for b in (1, batch // 2, batch):
        assert _default(h, w, direction, b) == few, b
    for b in (batch + 1, LARGE):
        assert _default(h, w, direction, b) == many, b
    assert dct.get_variant(h, w, direction, "fp32") == many


@pytest.mark.parametrize("h,w,direction,lo,hi", [(128, 64, 1, 400, 1024), (128, 64, 2, 560, 960), (128, 32, 1, 512, 1024),
                                                 (32, 128, 3, 800, 1024), (128, 16, 3, 800, 1024), (64, 128, 3, 700, 900)])
def test_arrays_that_fill_the_chip_once(h, w, direction, lo, hi):
    assert [_default(h, w, direction, b) for b in (1, lo - 1, lo, hi, hi + 1, LARGE)] == [2, 2, 0, 0, 2, 2]


@pytest.mark.parametrize("h,w", SHAPES)
def test_round_trip_and_filter_run_the_same_variant(h, w):
    """Multipliers of one give the round trip bit for bit, at every batch."""
    for b in list(range(1, 1300)) + [4095, 4096, 6143, 6144, LARGE]:
        assert _default(h, w, 2, b) == _default(h, w, 3, b), b
