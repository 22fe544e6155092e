"""GPU parity of the dense path (spconv_forward_dense, fp32 products on the matrix cores) against the
oracle, with the layer tolerance 1e-5 * sum|w*x| + 1e-6 per output (both paths
accumulate in fp32; only the order differs). Cases cover one to four waves per
workgroup, several channel tiles, partial channel tiles (K not a multiple of
32), odd C (the zero pad channel), several LDS chunks, one to eight 32-pixel
blocks per wave, 1x1 and 3x3 filters, pool, residual and zero-bordered
outputs. Every case prints its name and plan before touching the GPU.
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


def say(*a):
    print("[case]", *a, flush=True)


def check_close(gpu, ref, ab, what=""):
    gpu = np.asarray(gpu, np.float64)
    assert gpu.shape == ref.shape, (gpu.shape, ref.shape)
    err = np.abs(gpu - ref)
    bad = err > REL_TOL * ab + ABS_TOL
    assert not bad.any(), f"{what}: {int(bad.sum())} of {bad.size} outputs out of tolerance, max err {err.max():.3e}"


# N, C, K, H, W, R, density, pool, residual
CASES = [
    (1, 4, 8, 6, 7, 3, 0.5, False, False),
    (2, 5, 40, 9, 11, 3, 0.6, True, False),
    (1, 3, 33, 14, 14, 3, 1.0, False, True),
    (2, 7, 130, 5, 6, 1, 0.7, False, False),
    (1, 66, 16, 4, 30, 3, 0.4, True, True),
    (1, 2, 4, 2, 2, 3, 1.0, True, False),
    (1, 3, 16, 3, 224, 3, 0.5, False, False),
    (2, 17, 64, 30, 58, 3, 0.3, False, False),
    (4, 64, 64, 28, 28, 3, 0.5, True, False),
    (1, 130, 20, 7, 9, 3, 0.5, False, False),
    (3, 32, 96, 16, 16, 3, 0.2, False, True),
    (2, 9, 200, 12, 12, 3, 0.5, True, True),
]


def _layer(i):
    N, C, K, H, W, R, d, pool, _ = CASES[i]
    return synth.random_layer(8000 + i, N, C, K, H, W, R, R, 1, 1 if R == 3 else 0, d, True, pool, True, False)


def _dense_layer(sp, layer):
    N, C, H, W, K, R, S = layer.shape
    return sp.SparseConvLayer(layer.w, layer.mask, layer.bias, H, W, 1, layer.pad, True, layer.pool, path="dense")


@pytest.mark.parametrize("i", range(len(CASES)))
def test_dense_against_oracle(sp, i):
    import torch
    layer = _layer(i)
    N, C, H, W, K, R, S = layer.shape
    L = _dense_layer(sp, layer)
    use_res = CASES[i][8]
    res = np.random.default_rng(200 + i).uniform(-1, 1, (N, K, H, W)).astype(np.float32) if use_res else None
    say("dense", CASES[i], L.plan(N))
    xp = L.pad_input(torch.from_numpy(layer.x).cuda())
    kw = {}
    if use_res:
        kw = dict(residual=torch.from_numpy(np.pad(res, ((0, 0), (0, 0), (1, 1), (1, 1)))).cuda(), residual_pad=1)
    out = L.forward_padded(xp, **kw)
    torch.cuda.synchronize()
    ref, ab = oracle.conv(layer.x, layer.w, layer.mask, layer.bias, 1, layer.pad, True, layer.pool, residual=res)
    check_close(out.cpu().numpy(), ref, ab, f"dense {CASES[i]}")


@pytest.mark.parametrize("i", [0, 1, 7, 8])
def test_dense_out_pad_bitwise(sp, i):
    """A zero-bordered output holds the plain call's values bit for bit."""
    import torch
    layer = _layer(i)
    N, C, H, W, K, R, S = layer.shape
    L = _dense_layer(sp, layer)
    say("dense out_pad", CASES[i], L.plan(N))
    xp = L.pad_input(torch.from_numpy(layer.x).cuda())
    plain = L.forward_padded(xp)
    buf = torch.full((N, K, L.Ho + 2, L.Wo + 2), float("nan"), device="cuda")
    L.forward_padded(xp, out=buf, out_pad=1)
    torch.cuda.synchronize()
    ref = np.pad(plain.cpu().numpy(), ((0, 0), (0, 0), (1, 1), (1, 1)))
    assert np.array_equal(buf.cpu().numpy().view(np.uint32), ref.view(np.uint32))


def test_dense_full_size_narrow(sp):
    """The deep narrow layer at density 0.5 (32 x 256 x 14x14, Beta(2,5) row
    skew) in the plan the benchmark runs, whole output tensor against the
    oracle, and the dispatcher's choice for it."""
    import torch
    layer = synth.make_layer("narrow_d0.5")
    N, C, H, W, K, R, S = layer.shape
    L = sp.SparseConvLayer(layer.w, layer.mask, layer.bias, H, W, 1, 1, True, False, path="auto", N=N)
    assert L.path == "dense"
    say("dense narrow_d0.5 full size", L.plan(N))
    out = L.run(torch.from_numpy(layer.x).cuda())
    torch.cuda.synchronize()
    ref, ab = oracle.conv(layer.x, layer.w, layer.mask, layer.bias, 1, 1, True, False)
    check_close(out.cpu().numpy(), ref, ab, "narrow_d0.5 dense")


def test_dense_and_sparse_agree(sp):
    """Both paths on one layer (ResNet-shaped, small batch): each within the
    layer tolerance of the oracle."""
    import torch
    layer = synth.random_layer(77, 2, 64, 64, 56, 56, 3, 3, 1, 1, 0.3, True, False, True, False)
    N, C, H, W, K, R, S = layer.shape
    x = torch.from_numpy(layer.x).cuda()
    outs = {}
    for path in ("sparse", "dense"):
        L = sp.SparseConvLayer(layer.w, layer.mask, layer.bias, H, W, 1, 1, True, False, path=path)
        say("agree", path, L.plan(N))
        outs[path] = L.run(x)
    torch.cuda.synchronize()
    ref, ab = oracle.conv(layer.x, layer.w, layer.mask, layer.bias, 1, 1, True, False)
    for path, o in outs.items():
        check_close(o.cpu().numpy(), ref, ab, path)


# N, C, K, H, W, R, pool: channel counts around the 16-channel groups, K around
# the 32-channel tiles, one to eight pixel blocks shared by one to four waves
# (single rows and blocks past the last stored pixel among them).
GROUP_CASES = [
    (1, 1, 1, 3, 3, 3, False),
    (1, 15, 31, 5, 34, 3, False),
    (2, 16, 32, 9, 30, 3, True),
    (1, 17, 33, 2, 222, 3, False),
    (1, 33, 65, 8, 62, 3, True),
    (3, 48, 129, 7, 7, 3, False),
    (2, 8, 64, 6, 253, 3, False),
    (1, 40, 40, 12, 125, 3, True),
    (2, 31, 97, 11, 33, 1, False),
    (1, 130, 36, 10, 64, 1, True),
]


@pytest.mark.parametrize("case", GROUP_CASES)
def test_dense_channel_groups_and_unpadded_input(sp, case):
    """Against the oracle, and the unpadded input against the padded one bit for bit."""
    import torch
    N, C, K, H, W, R, pool = case
    layer = synth.random_layer(8100 + C, N, C, K, H, W, R, R, 1, R // 2, 0.6, True, pool, True, False)
    L = _dense_layer(sp, layer)
    say("dense groups", case, L.plan(N))
    x = torch.from_numpy(layer.x).cuda()
    out = L.run(x)
    raw = L.forward(x, pad_in_kernel=True)
    torch.cuda.synchronize()
    ref, ab = oracle.conv(layer.x, layer.w, layer.mask, layer.bias, 1, layer.pad, True, pool)
    check_close(out.cpu().numpy(), ref, ab, f"dense {case}")
    assert np.array_equal(out.cpu().numpy().view(np.uint32), raw.cpu().numpy().view(np.uint32))


def test_dense_extreme_values(sp):
    """Infinities, NaN and values that round to infinity in bf16 give what fp32
    arithmetic over every tap gives, and leave the other outputs alone; tiny
    values keep their leading bits."""
    import torch
    layer = synth.random_layer(8200, 2, 20, 40, 12, 13, 3, 3, 1, 1, 1.0, False, False, True, False)
    layer.w[layer.w == 0] = 0.5
    layer.w[3] *= 1e-6
    layer.x[0, 2, 4, 5] = np.inf
    layer.x[0, 7, 9, 9] = -np.inf
    layer.x[0, 1, 0, 12] = np.nan
    layer.x[1, 3, 6, 6] = 3.4028e38
    layer.x[1, 5, 2, 2] = 1e-30
    L = sp.SparseConvLayer(layer.w, layer.mask, layer.bias, 12, 13, 1, 1, False, False, path="dense")
    say("dense extreme values", L.plan(2))
    out = L.run(torch.from_numpy(layer.x).cuda())
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    with np.errstate(all="ignore"):
        ref = torch.nn.functional.conv2d(torch.from_numpy(layer.x).double(), torch.from_numpy(layer.w).double(),
                                         torch.from_numpy(layer.bias).double(), padding=1).numpy()
        ab = torch.nn.functional.conv2d(torch.from_numpy(np.abs(layer.x)).double(),
                                        torch.from_numpy(np.abs(layer.w)).double(), padding=1).numpy()
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    inf = np.isinf(ref)  # through an infinite input: float64 does not overflow here
    assert (ref[inf] > 0).any() and (ref[inf] < 0).any() and np.array_equal(got[inf], ref[inf])
    fin = np.isfinite(ref) & (ab < 3e38)  # (finite inputs may overflow fp32 beyond)
    assert np.isfinite(got[fin]).all()
    assert (np.abs(got[fin] - ref[fin]) <= REL_TOL * ab[fin] + ABS_TOL).all()


@pytest.mark.parametrize("C", [1, 3, 8])
@pytest.mark.parametrize("H,W,pool", [(5, 7, False), (17, 62, True), (4, 222, False), (12, 94, True)])
def test_dense_tap_pairs(sp, C, H, W, pool):
    """At most 8 channels: two taps to a matrix step (one to eight pixel blocks),
    against the oracle and with an infinite and a NaN input next to finite ones."""
    import torch
    layer = synth.random_layer(8300 + C, 2, C, 40, H, W, 3, 3, 1, 1, 0.8, False, pool, True, False)
    layer.w[:] = np.where(layer.w == 0, 0.25, layer.w)
    L = sp.SparseConvLayer(layer.w, None, layer.bias, H, W, 1, 1, False, pool, path="dense")
    say("dense tap pairs", C, H, W, pool, L.plan(2))
    x = torch.from_numpy(layer.x).cuda()
    out = L.run(x)
    padded = L.forward_padded(L.pad_input(x))
    bad = x.clone()
    bad[0, C - 1, 2, 3] = float("inf")
    bad[1, 0, 4 if H > 4 else 3, W - 1] = float("nan")
    raw = L.run(bad)
    torch.cuda.synchronize()
    ref, ab = oracle.conv(layer.x, layer.w, None, layer.bias, 1, 1, False, pool)
    check_close(out.cpu().numpy(), ref, ab, f"tap pairs {C} {H}x{W}")
    assert np.array_equal(out.cpu().numpy().view(np.uint32), padded.cpu().numpy().view(np.uint32))
    conv = torch.nn.functional.conv2d(bad.cpu().double(), torch.from_numpy(layer.w).double(),
                                      torch.from_numpy(layer.bias).double(), padding=1).numpy()
    touched = ~np.isfinite(conv)
    got, want, clean = raw.cpu().double().numpy(), conv, out.cpu().double().numpy()
    if pool:  # a window's maximum skips NaN, unless all four are
        def corners(t):
            t = t[:, :, :H // 2 * 2, :W // 2 * 2]
            return [t[:, :, i::2, j::2] for i in (0, 1) for j in (0, 1)]
        want = np.fmax.reduce(corners(conv))
        touched = np.logical_or.reduce(corners(touched))
    assert np.isinf(want).any()
    assert np.array_equal(np.isnan(got), np.isnan(want))
    assert np.array_equal(got[np.isinf(want)], want[np.isinf(want)])
    assert np.array_equal(got[~touched], clean[~touched])
    some = touched & np.isfinite(want)
    assert np.allclose(got[some], want[some], rtol=1e-5, atol=1e-5)


def test_dense_more_images_than_one_launch_counts(sp):
    """34 million images of 3x3 on 128 threads each pass the 2^32 threads of one
    launch: every image against the same image in calls of a million (bit for bit)."""
    import torch
    N, part = 34_000_000, 1_000_000
    layer = synth.random_layer(8400, 1, 1, 1, 3, 3, 3, 3, 1, 1, 1.0, True, False, True, False)
    L = _dense_layer(sp, layer)
    p = L.plan(N)
    assert p["launch_workgroups"] * p["threads_per_workgroup"] >= 1 << 32
    say("dense many images", p)
    g = torch.Generator(device="cuda").manual_seed(1)
    x = torch.randn((N, 1, 3, 3), generator=g, device="cuda")
    out = L.forward(x)
    for n in range(0, N, part):
        assert torch.equal(out[n:n + part], L.forward(x[n:n + part]))
    torch.cuda.synchronize()
    del x, out
    torch.cuda.empty_cache()


@pytest.mark.parametrize("C,K,H,W,pool", [(24, 40, 12, 13, False), (24, 72, 28, 30, True), (5, 40, 9, 30, False),
                                          (64, 33, 7, 7, False)])
def test_dense_results_near_the_top_of_the_range(sp, C, K, H, W, pool):
    """1.7e38 * 2 is finite; its bf16 part rounds up to 2^127, whose product with 2 is not."""
    import torch
    layer = synth.random_layer(8500 + C, 2, C, K, H, W, 3, 3, 1, 1, 1.0, False, pool, True, False)
    layer.w[:, 3, 1, 1] = 2.0
    layer.x[0, 3, 4, 5] = 1.7e38
    layer.x[1, 3, 2, 2] = -1.7e38
    layer.x[1, 3, 6, 6] = 3.4028e38  # rounds to infinity in bf16
    layer.w[0, 3, 1, 1] = 0.99
    L = sp.SparseConvLayer(layer.w, None, layer.bias, H, W, 1, 1, False, pool, path="dense")
    say("dense top of the range", L.plan(2))
    out = L.run(torch.from_numpy(layer.x).cuda())
    torch.cuda.synchronize()
    ref, ab = oracle.conv(layer.x, layer.w, None, layer.bias, 1, 1, False, pool)
    assert (np.abs(ref) > 3.3e38).any()
    with np.errstate(over="ignore"):
        want = ref.astype(np.float32).astype(np.float64)  # infinite where the sum is
    got = out.cpu().numpy().astype(np.float64)
    assert np.array_equal(got[np.isinf(want)], want[np.isinf(want)])
    fin = np.isfinite(want)
    assert (np.abs(got[fin] - want[fin]) <= REL_TOL * ab[fin] + ABS_TOL).all()


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_dense_input_without_a_finite_value(sp, value):
    """Every sum not finite (a diverged network): what fp32 gives on the CPU, for
    one, two and four reduction shares and tap pairs. (Taking these sums again
    one output at a time took hundreds of times a normal pass.)"""
    import torch
    for N, C, K, H, W, pool in [(2, 48, 64, 14, 14, False), (1, 40, 33, 9, 30, True), (2, 3, 40, 7, 9, False),
                                (64, 32, 128, 14, 14, False)]:
        layer = synth.random_layer(8600 + C, N, C, K, H, W, 3, 3, 1, 1, 1.0, False, pool, True, False)
        L = sp.SparseConvLayer(layer.w, None, layer.bias, H, W, 1, 1, False, pool, path="dense")
        say("dense", value, L.plan(N))
        x = torch.full((N, C, H, W), value)
        out = L.run(x.cuda()).cpu()
        raw = L.forward(x.cuda(), pad_in_kernel=True).cpu()
        assert torch.equal(torch.isnan(raw), torch.isnan(out)) and torch.equal(torch.nan_to_num(raw), torch.nan_to_num(out))
        ref = torch.nn.functional.conv2d(x[:1], torch.from_numpy(layer.w), torch.from_numpy(layer.bias), padding=1)
        assert not torch.isfinite(ref).any()
        if pool:  # a window's maximum skips NaN, unless all four are
            ref = torch.nan_to_num(ref, nan=-float("inf"), posinf=float("inf"), neginf=-float("inf"))
            assert not torch.isfinite(out).any()
            m = torch.nn.functional.max_pool2d(ref, 2)
            assert torch.equal(out == float("inf"), (m == float("inf")).expand_as(out))
            continue
        assert torch.equal(torch.isnan(out), torch.isnan(ref).expand_as(out))
        assert torch.equal(torch.nan_to_num(out), torch.nan_to_num(ref).expand_as(out))


@pytest.mark.parametrize("C,H,W,R", [(2, 2_100_000, 253, 3), (13, 620_000, 131, 1), (16, 230_000, 253, 3),
                                     (40, 200_000, 253, 3)])
def test_dense_tall_planes(sp, C, H, W, R):
    """Chunks near the end of 32-bit byte offsets (8 GB of input): bands of rows at the
    ends and between against float64, the rest finite and where the ReLU left it."""
    import torch
    K, pad = 2, R // 2
    layer = synth.random_layer(8700 + C, 1, C, K, 8, 8, R, R, 1, pad, 1.0, True, False, True, False)
    L = sp.SparseConvLayer(layer.w, None, layer.bias, H, W, 1, pad, True, False, path="dense")
    say("dense tall planes", C, H, W, L.plan(1))
    g = torch.Generator(device="cuda").manual_seed(C)
    x = torch.rand((1, C, H, W), generator=g, device="cuda")
    out = L.forward(x)
    torch.cuda.synchronize()
    w, b = torch.from_numpy(layer.w).double(), torch.from_numpy(layer.bias).double()
    for r0 in (0, H // 3, H // 2 + 7, H - 20):
        r1 = min(H, r0 + 20)
        lo, hi = max(0, r0 - pad), min(H, r1 + pad)
        band = torch.nn.functional.pad(x[:, :, lo:hi].cpu().double(),
                                       (pad, pad, pad - (r0 - lo), pad - (hi - r1)))
        ref = torch.relu(torch.nn.functional.conv2d(band, w, b))
        ab = torch.nn.functional.conv2d(band, w.abs(), b.abs())
        check_close(out[:, :, r0:r1].cpu().numpy(), ref.numpy(), ab.numpy(), f"rows {r0}..")
    assert bool((out >= 0).all()) and bool(torch.isfinite(out).all())
    del x, out
    torch.cuda.empty_cache()


@pytest.mark.parametrize("C", [5, 40])
@pytest.mark.parametrize("scale", [1e-32, 1e-34, 1e-35, 1e-36])
def test_dense_small_values(sp, C, scale):
    """Inputs of one magnitude down to 1e-36: below 2^-110 they count to the nearest
    multiple of 2^-133, an error of at most 2^-134 for each factor of the filter;
    above, relative errors are those of ordinary values."""
    import torch
    layer = synth.random_layer(8800 + C, 2, C, 40, 14, 14, 3, 3, 1, 1, 1.0, False, False, False, False)
    x = ((layer.x + 0.5) * np.float32(scale)).astype(np.float32)
    L = sp.SparseConvLayer(layer.w, None, None, 14, 14, 1, 1, False, False, path="dense")
    say("dense small values", C, scale, L.plan(2))
    out = L.run(torch.from_numpy(x).cuda())
    torch.cuda.synchronize()
    ref, ab = oracle.conv(x, layer.w, None, None, 1, 1, False, False)
    _, wsum = oracle.conv(np.ones_like(x), layer.w, None, None, 1, 1, False, False)
    lost = 2.0 ** -134 * wsum if scale < 2.0 ** -109 else 0.0
    assert (np.abs(out.cpu().numpy() - ref) <= 1e-6 * ab + lost).all()
