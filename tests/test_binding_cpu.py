"""CPU tests of the binding's host side: what a layer decides once, and what the
helpers of a forward call accept. Layers are built on the CPU; nothing is
queued on a GPU."""
import ctypes

import pytest

from paper_2005_04091_amd import synth


@pytest.fixture(scope="module")
def sp():
    from paper_2005_04091_amd import spconv
    return spconv


def _layer(sp, W, density, path="sparse", stride=1, pool=False):
    layer = synth.random_layer(W, 1, 128, 128, W, W, 3, 3, stride, 1, density, True, pool, True, False)
    return sp.SparseConvLayer(layer.w, layer.mask, layer.bias, W, W, stride, 1, True, pool, device="cpu", path=path)


@pytest.mark.parametrize("W,density,path,stride,want", [
    (14, 0.05, "sparse", 1, False),  # the walk on rows of no whole 16-byte groups
    (57, 0.05, "sparse", 1, False),
    (14, 0.9, "sparse", 1, True),    # the matrix kernel
    (16, 0.05, "sparse", 1, True),
    (14, 0.9, "dense", 1, True),
    (14, 0.2, "sparse", 2, False),   # strided
])
def test_pads_in_kernel_plans_once(sp, monkeypatch, W, density, path, stride, want):
    """The decision of a batch size and flags is made once: a second call asks no plan."""
    layer = _layer(sp, W, density, path, stride)
    asked = []
    plan = sp.spconv_plan
    monkeypatch.setattr(sp, "spconv_plan", lambda *a, **kw: asked.append(a[0]) or plan(*a, **kw))
    assert layer.pads_in_kernel(32) is want
    del asked[:]
    assert layer.pads_in_kernel(32) is want and not asked
    layer.pads_in_kernel(8)
    del asked[:]
    assert layer.pads_in_kernel(8) is layer.pads_in_kernel(8) and not asked


def test_output_shape_refuses_floats_it_has_answered_as_integers(sp):
    assert sp.spconv_output_shape(14, 14, 3, 3, 1, 1, 1) == (14, 14)
    for args in [(14.0, 14, 3, 3, 1, 1, 1), (14, 14, 3, 3, 1.0, 1, 1), (14, 14, 3, 3, 1, 1, 1.0)]:
        with pytest.raises(ctypes.ArgumentError):
            sp.spconv_output_shape(*args)


def test_forward_refuses_floats_for_remembered_sizes(sp):
    """The forward calls remember output shapes by value, and 14.0 equals 14: the
    library call refuses it (nothing is queued: the buffers are NULL too)."""
    assert sp._output_shape(14, 14, 3, 3, 1, 1, 1) == sp._output_shape(14.0, 14, 3, 3, 1, 1, 1)
    csr = sp.spconv_csr(4, 4, 3, 3, 16, 16, 0, None, None, None, None)
    with pytest.raises(ctypes.ArgumentError):
        sp._lib.spconv_forward_ex(None, 1, 4, 14.0, 14, ctypes.byref(csr), 4, 3, 3, 1, 1, None, 1, None, None, None)
