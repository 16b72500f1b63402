"""fp32 sums on the split bf16 products: what becomes of infinities, NaNs and very small numbers, how the error grows with
the length of a sum, and what a pass with an infinity in it costs.  References in fp64 on the device."""
import pytest
import torch

import paper_2006_03108_amd as dd
from tests.gpu_util import ConvLayer, require_gpu, split_forms

pytestmark = pytest.mark.gpu


def _rel(got, want):
    return float((got.double() - want).norm() / want.norm().clamp_min(1e-300))


# (batch, channels, extents, kernel, stride): gather kernels with 256 and 64 rows, patch kernels with one to three M-tiles,
# classes of a stride, several output planes per workgroup; the weight gradient of each
LAYERS = [(1, 5, 40, (24, 24), 7, 1), (12, 32, 32, (120, 116), 3, 1), (2, 18, 33, (40, 44), 3, 2), (1, 32, 32, (20, 22, 24), 5, 2),
          (3, 8, 64, (300,), 3, 1), (2, 60, 36, (37, 40), 3, 1), (2, 4, 4, (150, 140), 5, 1)]
IDS = ["x".join(map(str, v[3])) + f"c{v[1]}-{v[2]}s{v[5]}" for v in LAYERS]


@pytest.mark.parametrize("shape", LAYERS, ids=IDS)
def test_conv_with_infinities_and_nans(shape):
    """Every sum without such a term is as exact as ever, also those of the same tile and of the planes after it; every
    other one is the infinity or NaN that fp64 gives."""
    require_gpu()
    n_b, c_in, c_out, n, k, s = shape
    L = ConvLayer(*shape)
    inner, last = L.x[L.bulk], n_b - 1
    inner[(last, *(v // 2 for v in n), 1)], inner[(0, *(v - 1 for v in n), 0)] = float("inf"), float("nan")
    inner[(n_b // 2, *([3] * len(n)), c_in - 1)] = 3.0e38          # finite, and so are its products with 1e-3
    L.w[:, c_in - 1] *= 1e-3
    out = L.dy.shape[1:-1]
    L.dy[(last, *(v // 3 for v in out), c_out - 1)], L.dy[(0, *(v // 2 for v in out), 2)] = float("-inf"), float("nan")
    for run in L.ways():
        for name, got, want in zip(("y", "dx", "dw"), run(), L.exact()):
            if name == "dw":                                             # (3e38 times dy overflows in one order and not in another)
                got, want = got[:, :-1], want[:, :-1]
            sure = (want.abs() < 1e38) | ~torch.isfinite(want)           # (those next to the largest number may go either way)
            assert torch.equal(torch.isnan(got)[sure], torch.isnan(want)[sure]), name
            assert torch.equal((got == float("inf"))[sure], (want == float("inf"))[sure]), name
            assert torch.equal((got == float("-inf"))[sure], (want == float("-inf"))[sure]), name
            plain = want.abs() < 1e30
            assert bool(plain.any()) or name == "dw"
            if bool(plain.any()):
                assert _rel(got[plain], want[plain]) < 5e-6, name


@pytest.mark.parametrize("shape", LAYERS[:-1], ids=IDS[:-1])
def test_conv_with_a_weight_that_is_not_finite(shape):
    """A cell of dx that the weight's tap does not reach has no such term.  (The last layer's dx is not made of split
    products.)"""
    require_gpu()
    n_b, c_in, c_out, n, k, s = shape
    L = ConvLayer(*shape)
    L.w[(1, 2, *[0] * len(n))], L.w[(c_out - 1, 0, *[k - 1] * len(n))] = float("inf"), float("nan")
    L.w[(c_out // 2, 1, *[k // 2] * len(n))] = float("-inf")
    for run in L.ways():
        for name, got, want in zip(("y", "dx"), run(), L.exact()):
            assert torch.equal(torch.isnan(got), torch.isnan(want)), name
            assert torch.equal(got == float("inf"), want == float("inf")) and torch.equal(got == float("-inf"), want == float("-inf")), name
            plain = torch.isfinite(want)
            assert bool(plain.any()) and _rel(got[plain], want[plain]) < 5e-6, name


# few channels: several cells to a position (two, three; rows that end within one; strides; classes that are launches of
# their own), pairs of taps to a product, both; one to three dimensions.  (More cells, and several workers: the layers of
# few channels in test_gpu_layers.py.)
FEW = [(6, 8, 4, (28, 30, 45), 3, 2), (2, 3, 32, (120, 130), 7, 2), (3, 3, 40, (2000,), 7, 2), (2, 8, 36, (90, 100), 5, 2),
       (2, 40, 3, (260, 250), 3, 1), (1, 6, 20, (25, 30, 26), 4, 3), (4, 20, 8, (300, 280), 3, 1)]
FEW_IDS = ["x".join(map(str, v[3])) + f"c{v[1]}-{v[2]}s{v[5]}" for v in FEW]
# (cells to a position, products that two taps share) forward and in the data gradient, None on another kernel; by dilation
FEW_FORMS = {1: [(None, (2, 2)), (None, (1, 0)), (None, (1, 0)), (None, (1, 0)), ((3, 8), None), (None, (1, 0)), ((3, 8), (1, 0))],
             2: [(None, (2, 5)), (None, (1, 0)), (None, (1, 0)), ((1, 0), (1, 0)), ((1, 0), None), (None, (1, 0)), ((3, 11), (1, 0))]}


@pytest.mark.parametrize("dilation", [1, 2])
@pytest.mark.parametrize("shape", FEW, ids=FEW_IDS)
def test_layers_of_few_channels(shape, dilation):
    """Sums of at most 2000 products: 5e-6, as above."""
    require_gpu()
    L = ConvLayer(*shape, dil=dilation)
    assert split_forms(L.plan) == FEW_FORMS[dilation][FEW.index(shape)]
    for run in L.ways():
        L.y.fill_(7.0), L.dx.fill_(5.0)
        for name, got, want in zip(("y", "dx", "dw"), run(), L.exact()):
            assert _rel(got, want) < 5e-6, name
            assert float((got.double() - want).abs().max() / want.abs().max()) < 1e-5, name


@pytest.mark.parametrize("shape", FEW, ids=FEW_IDS)
def test_few_channels_with_infinities_and_nans(shape):
    """The zeros that fill up the weights of a position meet infinities that its cell has nothing to do with."""
    test_conv_with_infinities_and_nans(shape)


@pytest.mark.parametrize("shape", FEW, ids=FEW_IDS)
def test_few_channels_with_a_weight_that_is_not_finite(shape):
    test_conv_with_a_weight_that_is_not_finite(shape)


@pytest.mark.parametrize("c_in,c_out,n,k,s,p,fold", [(21840, 20, 40, 8, 2, 3, 2), (33000, 8, 17, 7, 2, 3, 1)])
def test_data_gradient_of_very_many_channels(c_in, c_out, n, k, s, p, fold):
    """43680 columns of a position, whose bounds fit 16 bits, and a layer that would have too many for that; sums of at most 320
    products."""
    require_gpu()
    L = ConvLayer(1, c_in, c_out, (n, n), k, s, p=p)
    assert dd.distdl_debug_conv_kernels(L.plan)[1] == 3 and dd.distdl_debug_conv_split(L.plan, True)[1] == fold
    L.dx.fill_(5.0)
    got, want = L.run()[1], L.exact()[1]
    assert _rel(got, want) < 5e-6 and float((got.double() - want).abs().max() / want.abs().max()) < 1e-5


def test_weights_of_more_blocks_than_a_launch_has_along_one_dimension():
    """64 classes of a stride, 2 GiB of weights: 16.9 million blocks of them.  Sums of 23232 products."""
    require_gpu()
    L = ConvLayer(1, 23232, 23232, (4, 4, 4), 1, 4)
    assert dd.distdl_debug_conv_kernels(L.plan)[:2] == (3, 3) and dd.distdl_debug_conv_split(L.plan, True)[0] == 64
    L.dx.fill_(5.0)
    for name, got, want in list(zip(("y", "dx"), L.run(), L.exact())):
        assert _rel(got, want) < 5e-6, name


@pytest.mark.parametrize("small", ["x", "w", "dy"])
@pytest.mark.parametrize("shape", LAYERS, ids=IDS)
def test_conv_of_very_small_numbers(shape, small):
    """Numbers around 1e-36 have as many bits as any other (a bf16 number below 2^-126 = 1.2e-38 has not): 5e-6 is the bound
    of the other tests, far above what these sums show with operands around 1."""
    require_gpu()
    L = ConvLayer(*shape)
    getattr(L, small).mul_(1e-36)
    for run in L.ways():
        for name, got, want in zip(("y", "dx", "dw"), run(), L.exact()):
            assert _rel(got, want) < 5e-6, name


@pytest.mark.parametrize("small", ["x", "W", "dy"])
@pytest.mark.parametrize("n_b,n_fi,n_fo", [(70, 100, 130), (256, 1024, 1024), (37, 333, 77), (256, 4096, 4096)])
def test_affine_of_very_small_numbers(n_b, n_fi, n_fo, small):
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(6)
    new = lambda *sh: torch.randn(sh, generator=g, device="cuda")
    t = dict(x=new(n_b, n_fi), W=new(n_fo, n_fi), dy=new(n_b, n_fo))
    t[small].mul_(1e-36)
    x, W, dy = t["x"], t["W"], t["dy"]
    y, dx, dW = torch.empty_like(dy), torch.empty_like(x), torch.empty_like(W)
    plan = dd.distdl_affine_plan_create(n_b, n_fi, n_fo, 1, 1)
    for route in (-1, 0):
        dd.distdl_debug_affine_route(plan, route)
        dd.distdl_affine_fwd(plan, [x], [W], None, [y])
        dd.distdl_affine_bwd(plan, [x], [W], [dy], [dx], [dW], None)
        for got, want in ((y, x.double() @ W.double().t()), (dx, dy.double() @ W.double()), (dW, dy.double().t() @ x.double())):
            assert _rel(got, want) < 1e-6


@pytest.mark.parametrize("shape", [(1, 64, 64, (18, 18, 18), 7, 1), (1, 36, 40, (60, 61), 15, 1)], ids=["7^3", "15^2"])
def test_long_sums_are_not_biased(shape):
    """21952 and 8100 products a sum.  fp32 MFMAs round a running sum once for two products: relative error (2-norm)
    sqrt(K / 2 / 2) roundings of up to 2^-24 of it, 4.4e-6 for the longer one, mean error zero.  The split sums stay below
    that, and their mean error is far below a rounding (a bf16 MFMA drops bits towards minus infinity: kept in one
    accumulator all its products gave -8e-7)."""
    require_gpu()
    L = ConvLayer(*shape)
    for name, got, want in zip(("y", "dx"), L.run(), L.exact()):
        diff = got.double() - want
        rms = float(want.square().mean().sqrt())
        assert abs(float(diff.mean())) < 1e-7 * rms, name
        assert _rel(got, want) < 4.4e-6, name


def test_affine_sums_are_not_biased():
    """16.8 million sums of 256 and 4096 products: the mean of their errors, each below 3e-7 of the rms and of either sign, is
    about 10^-10 of it; a bias of a twentieth of a rounding would be 3e-9."""
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(7)
    new = lambda *sh: torch.randn(sh, generator=g, device="cuda")
    x, W, dy = new(256, 4096), new(4096, 4096), new(256, 4096)
    y, dx, dW = torch.empty_like(dy), torch.empty_like(x), torch.empty_like(W)
    plan = dd.distdl_affine_plan_create(256, 4096, 4096, 1, 1)
    dd.distdl_affine_fwd(plan, [x], [W], None, [y])
    dd.distdl_affine_bwd(plan, [x], [W], [dy], [dx], [dW], None)
    for got, want in ((y, x.double() @ W.double().t()), (dx, dy.double() @ W.double()), (dW, dy.double().t() @ x.double())):
        diff, rms = got.double() - want, float(want.square().mean().sqrt())
        assert float(diff.norm() / want.norm()) < 3e-7
        assert abs(float(diff.mean())) < 3e-9 * rms


def _time(fn):
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    fn()
    best = float("inf")
    for _ in range(3):
        a.record()
        fn()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


def test_a_pass_with_nans_costs_what_fp32_products_do():
    """A tile that has to be made again takes fp32 MFMAs, at 6 / 16 of the rate, and a pass over NaNs alone makes every tile
    twice: 1 + 16 / 6 times a clean pass, and twice that is allowed for here.  One infinity touches a few tiles."""
    require_gpu()
    L = ConvLayer(2, 32, 32, (64, 64, 64), 3, 1)
    clean = _time(L.run)
    L.x[L.bulk][(0, 30, 30, 30, 5)] = float("inf")
    assert _time(L.run) < 3 * clean
    L.x.fill_(float("nan"))
    L.dy.fill_(float("nan"))
    assert _time(L.run) < 2 * (1 + 16 / 6) * clean
    assert bool(torch.isnan(L.dw).all()) and bool(torch.isnan(L.y).all())
