"""GPU parity of the matrix-core kernel for CSR filters (strided layers of eight
or more input channels) against the oracle, whole tensors at the layer tolerance
1e-5 * sum|w*x| + 1e-6. Its products are fp32 values as three bf16 parts with
fp32 sums, so the tolerance is that of the other kernels. Cases cover every
compiled instance, channel counts around the octets and chunks, output channels
around the 16-channel row blocks, strides 2 and 3, filters of 1x1 to 7x7 and
unequal sides, rows of several tiles, empty and full filters, and rows with more
entries per chunk than the prefetched queue holds. Every case prints its name
and plan before touching the GPU.
"""
import numpy as np
import pytest

import oracle
from paper_2005_04091_amd import synth

pytestmark = pytest.mark.gpu

REL_TOL = 1e-5
ABS_TOL = 1e-6


@pytest.fixture(scope="module")
def sp():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2005_04091_amd import spconv
    return spconv


def check_close(got, ref, ab, what):
    got = np.asarray(got, np.float64)
    assert got.shape == ref.shape, (got.shape, ref.shape)
    bad = ~(np.abs(got - ref) <= REL_TOL * ab + ABS_TOL)
    assert not bad.any(), f"{what}: {int(bad.sum())} of {bad.size} outputs out of tolerance"


# N, C, K, H, W, R, S, stride, pad, density, pool, skew
CASES = [
    (3, 8, 55, 6, 5, 1, 1, 3, 0, 0.1, False, False),      # (2 pixel blocks, 16 channels)
    (5, 25, 9, 6, 7, 7, 7, 3, 3, 0.05, True, False),
    (8, 8, 29, 96, 77, 1, 1, 2, 0, 0.2, False, False),    # (4, 16)
    (2, 10, 146, 50, 67, 1, 1, 2, 0, 0.2, True, False),
    (14, 8, 214, 62, 53, 1, 1, 2, 0, 0.29, False, False),  # (4, 32)
    (23, 59, 167, 41, 52, 1, 1, 2, 0, 0.06, True, False),
    (30, 13, 239, 27, 18, 1, 1, 2, 0, 0.06, False, False),  # (7, 16)
    (5, 9, 8, 186, 193, 3, 3, 2, 1, 0.1, True, False),
    (1, 8, 1, 3, 3, 3, 3, 2, 1, 1.0, False, False),       # smallest
    (2, 9, 16, 7, 9, 3, 3, 2, 1, 0.5, False, False),
    (2, 15, 17, 8, 8, 3, 3, 2, 0, 0.3, True, False),
    (1, 16, 31, 9, 31, 3, 1, 2, 1, 0.4, False, False),
    (1, 17, 33, 31, 9, 1, 3, 2, 1, 0.4, False, False),
    (2, 33, 65, 20, 21, 5, 5, 2, 2, 0.2, False, True),
    (1, 24, 40, 12, 300, 3, 3, 2, 1, 0.2, False, False),  # rows of several tiles
    (1, 24, 24, 31, 33, 3, 3, 3, 1, 0.0, False, False),   # no entries: act(bias)
    (2, 130, 20, 13, 14, 3, 3, 2, 1, 1.0, True, False),   # more entries per chunk than the queue
    (4, 64, 128, 56, 56, 3, 3, 2, 1, 0.2, False, False),
    (2, 40, 70, 33, 47, 3, 3, 4, 2, 0.3, False, True),
]


def _layer(i):
    N, C, K, H, W, R, S, st, pad, d, pool, skew = CASES[i]
    return synth.random_layer(9500 + i, N, C, K, H, W, R, S, st, pad, d, True, pool, i % 3 != 2, skew)


def _on_device(sp, layer):
    N, C, H, W, K, R, S = layer.shape
    L = sp.SparseConvLayer(layer.w, layer.mask, layer.bias, H, W, layer.stride, layer.pad, True, layer.pool)
    plan = L.plan(N)
    print("[case]", layer.shape, layer.stride, plan, flush=True)
    assert plan["kernel"] == sp.SPCONV_KERNEL_MATRIX
    return L, plan


@pytest.mark.parametrize("i", range(len(CASES)))
def test_strided_layers_and_epilogue_options(sp, i):
    import torch
    layer = _layer(i)
    N, C, H, W, K, R, S = layer.shape
    L, _ = _on_device(sp, layer)
    xp = L.pad_input(torch.from_numpy(layer.x).cuda())
    out = L.forward_padded(xp)
    res = np.random.default_rng(i).uniform(-1, 1, (N, K, (H + 2 * layer.pad - R) // layer.stride + 1,
                                                   (W + 2 * layer.pad - S) // layer.stride + 1)).astype(np.float32)
    res_dev = torch.from_numpy(np.pad(res, ((0, 0), (0, 0), (1, 1), (1, 1)))).cuda()
    buf = torch.full((N, K, L.Ho + 4, L.Wo + 4), float("nan"), device="cuda")
    L.forward_padded(xp, out=buf, out_pad=2, residual=res_dev, residual_pad=1)
    torch.cuda.synchronize()
    ref, ab = oracle.conv(layer.x, layer.w, layer.mask, layer.bias, layer.stride, layer.pad, True, layer.pool)
    check_close(out.cpu().numpy(), ref, ab, f"{CASES[i]}")
    ref, ab = oracle.conv(layer.x, layer.w, layer.mask, layer.bias, layer.stride, layer.pad, True, layer.pool,
                          residual=res)
    got = buf.cpu().numpy()
    check_close(got[:, :, 2:-2, 2:-2], ref, ab, f"{CASES[i]} residual")
    got[:, :, 2:-2, 2:-2] = 0
    assert not got.view(np.uint32).any(), "the border holds something else than +0.0"


def test_every_instance_has_a_case(sp):
    have = {(p["pixels_per_lane"], 0, p["channels_per_wave"], int(_layer(i).pool))
            for i in range(len(CASES)) for p in [_on_device(sp, _layer(i))[1]]}
    assert have == set(sp.spconv_kernel_variants(sp.SPCONV_KERNEL_MATRIX))


def test_extreme_values_touch_only_the_outputs_that_read_them(sp):
    """Infinities, NaN and values that round to infinity in bf16: each output is
    what its own entries give in fp32 (a zero of the filter reads nothing)."""
    import torch
    layer = synth.random_layer(9600, 2, 20, 40, 21, 23, 3, 3, 2, 1, 0.3, False, False, True, False)
    layer.x[0, 2, 4, 5] = np.inf
    layer.x[0, 7, 9, 9] = -np.inf
    layer.x[0, 1, 0, 12] = np.nan
    layer.x[1, 3, 6, 6] = 3.4028e38
    L, _ = _on_device(sp, layer)
    L.flags = 0  # no ReLU, which hides NaN and negative infinities
    out = L.forward_padded(L.pad_input(torch.from_numpy(layer.x).cuda()))
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    K = layer.w.shape[0]
    xp = np.pad(layer.x.astype(np.float64), ((0, 0), (0, 0), (1, 1), (1, 1)))
    ref = np.repeat(np.repeat(layer.bias.astype(np.float64)[None, :, None, None], L.Ho, 2), L.Wo, 3).repeat(2, 0)
    ab = np.zeros_like(ref)
    with np.errstate(all="ignore"):
        for k in range(K):
            for c, r, s in np.argwhere(layer.mask[k]):
                v = xp[:, c, r:r + 2 * L.Ho - 1:2, s:s + 2 * L.Wo - 1:2]
                ref[:, k] += layer.w[k, c, r, s] * v
                ab[:, k] += np.abs(layer.w[k, c, r, s] * v)
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    inf = np.isinf(ref)  # through an infinite input: float64 does not overflow here
    assert (ref[inf] > 0).any() and (ref[inf] < 0).any() and np.array_equal(got[inf], ref[inf])
    fin = np.isfinite(ref) & (ab < 3e38)  # (finite inputs may overflow fp32 beyond)
    assert np.isfinite(got[fin]).all()
    assert (np.abs(got[fin] - ref[fin]) <= REL_TOL * ab[fin] + ABS_TOL).all()
    assert fin.sum() > 0.7 * fin.size


def test_replayed_graph_matches_the_eager_call(sp):
    import torch
    layer = _layer(17)
    L, _ = _on_device(sp, layer)
    xp = L.pad_input(torch.from_numpy(layer.x).cuda())
    eager = L.forward_padded(xp).clone()
    out = torch.empty_like(eager)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        L.forward_padded(xp, out=out, stream=torch.cuda.current_stream())
    for _ in range(3):
        out.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int32), eager.view(torch.int32))


# N, C, K, H, W, R, density, pool: stride-1 layers the planner gives to the matrix kernel
STRIDE1 = [
    (8, 128, 128, 28, 28, 3, 0.6, True),
    (1, 256, 256, 14, 14, 3, 0.3, False),
    (2, 120, 100, 30, 41, 5, 0.4, False),
    (3, 200, 203, 20, 23, 3, 0.5, False),
]


@pytest.mark.parametrize("case", STRIDE1)
def test_stride1_layers(sp, case):
    """Against the oracle; an unpadded input gives the padded one's bits; a call
    with a lowered stream still runs the stride-1 kernel; the row hint changes
    nothing."""
    import torch
    N, C, K, H, W, R, d, pool = case
    layer = synth.random_layer(9700 + H, N, C, K, H, W, R, R, 1, R // 2, d, True, pool, True, False)
    L, _ = _on_device(sp, layer)
    x = torch.from_numpy(layer.x).cuda()
    assert L.pads_in_kernel(N) and L.lowered(N) is None
    out = L.run(x)
    raw = L.forward(x)
    args = (L.pad_input(x), N, C, H, W, L.csr, K, R, R, 1, L.pad, L.bias, L.flags)
    hinted = sp.spconv_forward(*args)
    lw = torch.from_numpy(sp.spconv_pack_lowered(L.host_csr, N, H, W, 1, L.pad, L.flags, L.csr.max_row_nnz)).cuda()
    walked = sp.spconv_forward_ex(*args, lowered=lw)
    torch.cuda.synchronize()
    ref, ab = oracle.conv(layer.x, layer.w, layer.mask, layer.bias, 1, layer.pad, True, pool)
    for what, t in (("matrix", out), ("lowered", walked)):
        check_close(t.cpu().numpy(), ref, ab, f"{what} {case}")
    assert torch.equal(out.view(torch.int32), raw.view(torch.int32))
    assert torch.equal(out.view(torch.int32), hinted.view(torch.int32))


@pytest.mark.parametrize("stride", [7, 1431655766, (1 << 31) - 1])
@pytest.mark.parametrize("C,H,W,R,S", [(8, 3, 3, 3, 3), (17, 5, 4, 5, 3), (16, 4, 6, 1, 3)])
def test_strides_past_the_plane(sp, stride, C, H, W, R, S):
    """One output pixel per image, against the oracle."""
    import torch
    layer = synth.random_layer(9800 + C, 3, C, 21, H, W, R, S, stride, 0, 0.4, True, False, True, False)
    L, plan = _on_device(sp, layer)
    assert (L.Ho, L.Wo, plan["tile_pixels"]) == (1, 1, 1)
    out = L.forward_padded(L.pad_input(torch.from_numpy(layer.x).cuda()))
    torch.cuda.synchronize()
    ref, ab = oracle.conv(layer.x, layer.w, layer.mask, layer.bias, stride, 0, True, False)
    check_close(out.cpu().numpy(), ref, ab, f"stride {stride}")


def test_results_near_the_top_of_the_range(sp):
    """1.7e38 * 2 is finite; its bf16 part rounds up to 2^127, whose product with 2
    is not. A value that rounds to infinity in bf16, times 0.99, is finite too."""
    import torch
    for pool in (False, True):
        layer = synth.random_layer(9900, 2, 24, 40, 21, 23, 3, 3, 2, 1, 0.3, False, pool, True, False)
        layer.mask[:, 3, 1, 1] = 1
        layer.w[:, 3, 1, 1] = 2.0
        layer.w[0, 3, 1, 1] = 0.99
        layer.x[0, 3, 4, 6] = 1.7e38
        layer.x[1, 3, 2, 2] = -1.7e38
        layer.x[1, 3, 6, 6] = 3.4028e38
        L, _ = _on_device(sp, layer)
        L.flags &= ~sp.SPCONV_RELU
        out = L.forward_padded(L.pad_input(torch.from_numpy(layer.x).cuda()))
        torch.cuda.synchronize()
        ref, ab = oracle.conv(layer.x, layer.w, layer.mask, layer.bias, 2, 1, False, pool)
        with np.errstate(over="ignore"):
            want = ref.astype(np.float32).astype(np.float64)
        assert (np.abs(want[np.isfinite(want)]) > 3.3e38).any()
        got = out.cpu().numpy().astype(np.float64)
        assert np.array_equal(got[np.isinf(want)], want[np.isinf(want)])
        fin = np.isfinite(want)
        assert (np.abs(got[fin] - want[fin]) <= REL_TOL * ab[fin] + ABS_TOL).all()


@pytest.mark.parametrize("value", [float("inf"), -float("inf"), float("nan")])
@pytest.mark.parametrize("i", [1, 4, 6, 12, 15, 16])
def test_input_without_a_finite_value(sp, i, value):
    """Every sum not finite (a diverged network), whole rows of entries taken again
    in fp32: what the entries' signs give. (Taking these sums again one output
    at a time took a hundred times a normal pass.)"""
    import torch
    layer = _layer(i)
    L, _ = _on_device(sp, layer)
    L.flags = 0
    N, C, H, W, K, R, S = layer.shape
    x = np.full(layer.x.shape, value, np.float32)
    out = L.forward_padded(L.pad_input(torch.from_numpy(x).cuda())).cpu().numpy()
    xp = np.pad(x[:1], ((0, 0), (0, 0), (layer.pad,) * 2, (layer.pad,) * 2))
    st, (Ho, Wo) = layer.stride, out.shape[2:]
    bias = np.zeros(K, np.float32) if layer.bias is None else layer.bias
    ref = np.repeat(np.repeat(bias[None, :, None, None], Ho, 2), Wo, 3)
    with np.errstate(all="ignore"):
        for k in range(K):
            for c, r, s in np.argwhere(layer.mask[k]):
                ref[:, k] += layer.w[k, c, r, s] * xp[:, c, r:r + st * Ho - st + 1:st, s:s + st * Wo - st + 1:st]
    fin = np.isfinite(ref)
    for n in range(N):
        assert np.array_equal(out[n][~fin[0]], ref[0][~fin[0]], equal_nan=True)
        assert np.allclose(out[n][fin[0]], ref[0][fin[0]], rtol=1e-5, atol=1e-6)


@pytest.mark.parametrize("side", ["inputs", "filter"])
@pytest.mark.parametrize("scale", [1e-32, 1e-34, 1e-35, 1e-36])
def test_small_values(sp, scale, side):
    """Inputs or filter values of one magnitude down to 1e-36: below 2^-110 they
    count to the nearest multiple of 2^-133, an error of at most 2^-134 for each
    factor of the other side; above, relative errors are those of ordinary values."""
    import torch
    layer = synth.random_layer(9950, 2, 40, 40, 21, 23, 3, 3, 2, 1, 0.3, False, False, False, False)
    x, w = layer.x + np.float32(0.5), layer.w + np.sign(layer.w) * np.float32(0.5)
    if side == "inputs":
        x = (x * np.float32(scale)).astype(np.float32)
    else:
        w = (w * np.float32(scale)).astype(np.float32)
    L = sp.SparseConvLayer(w, layer.mask, None, 21, 23, 2, 1, False, False)
    print("[case]", scale, side, L.plan(2), flush=True)
    assert L.plan(2)["kernel"] == sp.SPCONV_KERNEL_MATRIX
    out = L.forward_padded(L.pad_input(torch.from_numpy(x).cuda()))
    torch.cuda.synchronize()
    ref, ab = oracle.conv(x, w, layer.mask, None, 2, 1, False, False)
    one = (np.ones_like(x), w) if side == "inputs" else (x, np.where(layer.mask, np.float32(1), np.float32(0)))
    _, other = oracle.conv(*one, layer.mask, None, 2, 1, False, False)
    lost = 2.0 ** -134 * other if scale < 2.0 ** -109 else 0.0
    assert (np.abs(out.cpu().numpy() - ref) <= 1e-6 * ab + lost).all()


@pytest.mark.parametrize("case", STRIDE1)
def test_stride1_sums_that_are_not_finite(sp, case):
    """A few infinite and NaN pixels: the unpadded input gives the padded one's bits,
    and both what the stride-1 kernel gives (which multiplies no zero of the filter)."""
    import torch
    N, C, K, H, W, R, d, pool = case
    layer = synth.random_layer(9700 + H, N, C, K, H, W, R, R, 1, R // 2, d, False, pool, True, False)
    L, _ = _on_device(sp, layer)
    x = torch.from_numpy(layer.x).cuda()
    rng = np.random.default_rng(H)
    for v in (float("inf"), -float("inf"), float("nan"), 3.4028e38):
        x[rng.integers(N), rng.integers(C), rng.integers(H), rng.integers(W)] = v
    x[N - 1, C - 1, H - 1, W - 1] = float("inf")
    out, raw = L.run(x), L.forward(x)
    lw = torch.from_numpy(sp.spconv_pack_lowered(L.host_csr, N, H, W, 1, L.pad, L.flags, L.csr.max_row_nnz)).cuda()
    walked = sp.spconv_forward_ex(L.pad_input(x), N, C, H, W, L.csr, K, R, R, 1, L.pad, L.bias, L.flags, lowered=lw)
    torch.cuda.synchronize()
    assert torch.equal(torch.isnan(out), torch.isnan(raw)) and torch.equal(torch.nan_to_num(out), torch.nan_to_num(raw))
    assert not torch.isfinite(walked).all()
    assert torch.equal(torch.isnan(out), torch.isnan(walked)) and torch.equal(torch.isinf(out), torch.isinf(walked))
    inf = torch.isinf(walked)
    assert torch.equal(out[inf], walked[inf])
    fin = torch.isfinite(walked) & (walked.abs() < 1e30)
    # (well within 1e-5 of the sum of |w * x|, up to some 500 products of order 1 here)
    assert torch.allclose(out[fin], walked[fin], rtol=1e-4, atol=1e-3)
