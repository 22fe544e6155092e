"""CPU tests of what the benchmark reports about a layer's kernel."""
import pytest

import bench
from paper_2005_04091_amd import synth


@pytest.mark.parametrize("density,stride,path,family", [
    (0.05, 1, "sparse", "fwd"), (0.9, 1, "sparse", "matrix"), (0.2, 2, "sparse", "matrix"), (0.9, 1, "dense", "dense")])
def test_kernel_family(density, stride, path, family):
    from paper_2005_04091_amd import spconv
    layer = synth.random_layer(3, 1, 64, 64, 28, 28, 3, 3, stride, 1, density, True, False, True, False)
    L = spconv.SparseConvLayer(layer.w, layer.mask, layer.bias, 28, 28, stride, 1, device="cpu", path=path)
    assert bench.kernel_family(L, 32) == family
    assert len(bench.kernel_source_sha(family)) == 16
