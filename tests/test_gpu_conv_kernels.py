"""Each kernel of the convolution layer at shapes where the library picks it: the tiers that take what the split and gather
kernels do not (strides beyond theirs here, tensors of 2 GiB and more in earnest), and the weight gradients of the 16-wide
and of the bf16 tiles, which small layers do not reach.  Against fp64 on the device, by the bars of the other parity tests."""
import gc

import pytest
import torch

import paper_2006_03108_amd as dd
from tests.gpu_util import ConvLayer, require_gpu

pytestmark = pytest.mark.gpu
F32, BF16 = torch.float32, torch.bfloat16
TOL = {F32: 1e-5, BF16: 2e-2}

# (kernels of the forward pass, data gradient, weight gradient: 0 direct, 1 32-wide tiles, 2 16-wide tiles, 3 split, 4 gather),
# batch, channels, extents, kernel, stride, padding, dilation, type, elements into the allocation
CASES = [
    # direct kernels, both types, aligned or not; the weight gradient's operands read from memory (3, 5, 8 taps in a row)
    ((0, 0, 0), 2, 17, 19, (60, 66), (9, 9), (9, 9), 0, 1, F32, 0),
    ((0, 0, 0), 1, 3, 4, (61, 65), (9, 9), (9, 9), 4, 1, F32, 1),
    ((0, 0, 0), 2, 32, 32, (60, 66), (3, 3), (9, 9), 1, 1, BF16, 0),
    ((0, 0, 0), 1, 5, 7, (50, 49), (4, 5), (9, 9), 0, (1, 2), BF16, 1),
    ((0, 0, 1), 2, 32, 32, (60, 66), (3, 3), (9, 9), 0, 1, F32, 0),
    ((0, 0, 1), 2, 17, 19, (60, 66), (5, 5), (9, 9), 0, 1, F32, 0),
    ((2, 2, 1), 1, 3, 4, (60, 66), (7, 7), (9, 9), 0, 1, F32, 1),
    # fp32 32-wide tiles, one launch for each of up to 108 classes; the weight gradient staged in LDS (3 and 5 taps in a row)
    ((1, 1, 1), 1, 32, 36, (30, 31, 40), (2, 2, 3), (9, 9, 1), (0, 0, 1), 1, F32, 0),
    ((1, 1, 1), 1, 20, 8, (30, 31, 44), (2, 2, 5), (9, 9, 2), (0, 0, 2), 1, F32, 0),
    ((1, 1, 1), 1, 8, 24, (42, 50, 54), (2, 2, 3), (9, 3, 4), 0, 1, F32, 0),
    ((1, 1, 3), 1, 40, 36, (46, 43, 50), (3, 3, 3), (9, 2, 4), 1, 1, F32, 0),
    ((1, 1, 4), 1, 32, 32, (60, 64), (3, 3), (1, 1), 12, 12, F32, 0),
    # 16-wide weight gradient: aligned and not, one dimension, odd channels
    ((2, 2, 2), 2, 16, 16, (192, 224), (3, 3), (1, 1), 1, 1, F32, 0),
    ((2, 2, 2), 24, 16, 12, (36, 42), (3, 3), (1, 1), 1, 1, F32, 1),
    ((2, 2, 2), 24, 13, 16, (36, 42), (3, 3), (1, 1), 1, 1, F32, 0),
    ((2, 2, 2), 1, 4, 8, (48, 56), (1, 1), (1, 1), 0, 1, F32, 0),
    ((2, 2, 2), 16, 16, 16, (300,), (3,), (1,), 1, 1, F32, 0),
    # bf16 weight gradient, a kernel plane per workgroup: 9, 16 and 25 taps, row strides of 1 and 2, several channel tiles
    ((1, 1, 1), 1, 64, 64, (96, 112), (3, 3), (1, 1), 1, 1, BF16, 0),
    ((1, 1, 1), 6, 8, 24, (144, 168), (3, 3), (2, 2), 1, 1, BF16, 0),
    ((1, 1, 1), 1, 64, 64, (72, 84), (4, 4), (1, 1), 2, 1, BF16, 0),
    ((1, 1, 1), 1, 64, 64, (144, 168), (4, 4), (2, 2), 2, 1, BF16, 0),
    ((1, 1, 1), 1, 64, 64, (48, 56), (5, 5), (1, 1), 2, 1, BF16, 0),
    ((1, 1, 1), 1, 64, 64, (96, 112), (5, 5), (2, 2), 2, 1, BF16, 0),
    ((1, 1, 1), 1, 32, 32, (24, 28, 34), (3, 5, 5), (2, 2, 2), (1, 2, 2), 1, BF16, 0),
    ((1, 1, 1), 1, 32, 32, (36, 42, 51), (2, 4, 4), (1, 1, 1), (1, 2, 2), 1, BF16, 0),
]


@pytest.mark.parametrize("case", CASES, ids=[f"{c[2]}-{c[3]}k{'x'.join(map(str, c[5]))}s{'x'.join(map(str, c[6]))}{str(c[9])[6:]}o{c[10]}" for c in CASES])
def test_conv_kernel_against_fp64(case):
    require_gpu()
    want_kernels, n_b, c_in, c_out, shape, k, s, p, dil, dtype, offset = case
    L = ConvLayer(n_b, c_in, c_out, shape, k, s, dtype, p, dil, offset)
    assert dd.distdl_debug_conv_kernels(L.plan, aligned=offset == 0) == want_kernels
    L.y.fill_(7.0), L.dx.fill_(5.0), L.dw.fill_(9.0), L.db.fill_(9.0)
    exact = L.exact()
    for run in L.ways():
        for name, got, want in zip(("y", "dx", "dw"), run(), exact):
            diff = got.double() - want
            assert float(diff.norm() / want.norm()) < TOL[dtype], name
            assert float(diff.abs().max() / want.abs().max()) < TOL[dtype], name
        db = L.dy.double().reshape(-1, c_out).sum(0)
        assert float((L.db.double() - db).norm() / db.norm()) < TOL[dtype]


# where the choice among the fp32 kernels lies: planes of a few cells (gather), a class of a stride each (split), full windows
CHOICE = [((4, 4), 60, 36, 24, (5, 4, 3), (3, 3, 3), (1, 1, 1)), ((4, 3), 1, 8, 64, (5, 6, 9), (3, 3, 3), (2, 2, 2)),
          ((2, 3), 8, 2, 12, (180, 120), (3, 3), (2, 2)), ((3, 3), 2, 36, 40, (90, 91), (3, 3), (1, 1))]


@pytest.mark.parametrize("case", CHOICE, ids=[f"{c[2]}-{c[3]}" for c in CHOICE])
def test_choice_among_fp32_kernels(case):
    """Sums of at most 972 products, each within the bar of the other parity tests; and the same for tensors that are not
    aligned, which the split kernels do not take."""
    require_gpu()
    want_kernels, n_b, c_in, c_out, shape, k, s = case
    for offset in (0, 1):
        L = ConvLayer(n_b, c_in, c_out, shape, k, s, offset=offset)
        got_kernels = dd.distdl_debug_conv_kernels(L.plan, aligned=offset == 0)[:2]
        assert got_kernels == want_kernels if offset == 0 else 3 not in got_kernels
        for run in L.ways():
            for name, got, want in zip(("y", "dx"), run(), L.exact()):
                assert float((got.double() - want).norm() / want.norm()) < TOL[F32], name


# weight gradient of the gather kernel, 1, 63, 64, 65, 126, 128 and 129 rows (taps x input channels), with one and two column tiles,
# positions that end within an octet, a stage and a chunk, several workers' worth of chunks; before each case the rows of its tiles in
# fp32 and bf16 (0: the 16 x 16 kernel takes it)
FEW_ROWS = [((0, 256), 1, 1, 4, (33,), 1, 1), ((64, 256), 1, 1, 20, (33,), 1, 1), ((64, 64), 1, 1, 20, (5001,), 1, 1),
            ((64, 64), 3, 7, 33, (61, 47), 3, 1), ((64, 256), 1, 64, 5, (333,), 1, 1), ((64, 64), 1, 64, 5, (3333,), 1, 1),
            ((64, 64), 2, 13, 40, (129,), 5, 2), ((64, 64), 2, 14, 3, (50, 41), 3, 1), ((64, 64), 5, 16, 32, (9, 10, 11), 2, 1),
            ((64, 256), 2, 43, 64, (127,), 3, 1), ((64, 64), 2, 43, 64, (1271,), 3, 1), ((256, 256), 2, 43, 32, (127,), 3, 1),
            ((64, 64), 40, 3, 8, (90, 70), 3, 1)]


@pytest.mark.parametrize("offset", [0, 1], ids=["aligned", "odd"])
@pytest.mark.parametrize("dtype", [F32, BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("case", FEW_ROWS, ids=[f"{c[2] * c[5] ** len(c[4])}rows{c[3]}cols{c[4][0]}" for c in FEW_ROWS])
def test_weight_gradient_of_few_rows(case, dtype, offset):
    """fp32: a sum of n positions in chunks is off by at most sqrt(n / 16) roundings of 2^-24: 252 000 positions 7e-6."""
    require_gpu()
    rows, case = case[0][dtype == BF16], case[1:]
    L = ConvLayer(*case, dtype, offset=offset)
    assert dd.distdl_debug_conv_kernels(L.plan, offset == 0)[2] == (4 if rows else 2)
    assert not rows or dd.distdl_debug_conv_wgrad_rows(L.plan) == rows
    clean = L.dy[(0, *[0] * L.D, 1)].clone()
    for run in L.ways():
        L.dw.fill_(9.0), L.db.fill_(9.0), L.dy[(0, *[0] * L.D, 1)].copy_(clean)
        got, want = run()[2], L.exact()[2]
        assert float((got.double() - want).norm() / want.norm()) < TOL[dtype]
        assert float((got.double() - want).abs().max() / want.abs().max()) < TOL[dtype]
        db = L.dy.double().reshape(-1, case[2]).sum(0)
        assert float((L.db.double() - db).norm() / db.norm()) < TOL[dtype]
        if dtype == F32:  # an infinity stays with its rows and columns
            L.dy[(0, *[0] * L.D, 1)] = float("inf")
            got, want = run()[2], L.exact()[2]
            sure = torch.isfinite(want)
            assert torch.equal(torch.isfinite(got), sure)
            assert not bool(sure.any()) or float((got[sure].double() - want[sure]).norm() / want[sure].norm().clamp_min(1e-300)) < TOL[dtype]


# the same for bf16: planes of a few cells, classes of a stride, channels that are no multiples of 8, large layers
CHOICE_BF16 = [((4, 4), 9, 44, 36, (4, 4, 4), 3, 1), ((4, 4), 4, 4, 16, (150, 150), 5, 2), ((4, 4), 6, 12, 44, (60, 67), 3, 1),
               ((1, 4), 2, 56, 4, (54, 57, 62), 3, 1), ((1, 1), 10, 32, 8, (120, 110), 3, 1)]


@pytest.mark.parametrize("case", CHOICE_BF16, ids=[f"{c[2]}-{c[3]}" for c in CHOICE_BF16])
def test_choice_among_bf16_kernels(case):
    require_gpu()
    want_kernels, n_b, c_in, c_out, shape, k, s = case
    for offset in (0, 1):
        L = ConvLayer(n_b, c_in, c_out, shape, k, s, BF16, offset=offset)
        assert dd.distdl_debug_conv_kernels(L.plan, aligned=offset == 0)[:2] == (want_kernels if offset == 0 else (4, 4))
        for run in L.ways():
            for name, got, want in zip(("y", "dx"), run(), L.exact()):
                assert float((got.double() - want).norm() / want.norm()) < TOL[BF16], name


# 16 x 16 tiles: channel quads full and not (the patch's padding), 9, 25 and other tap counts, kernel planes, runs of a
# workgroup over several windows, samples stacked in a window, and fewer steps than workgroups
SIXTEEN = [(3, 4, 8, (90, 70), 3, 1), (2, 8, 16, (61, 83), 5, 1), (40, 16, 16, (70, 90), 3, 1), (2, 13, 5, (64, 64), 3, 1), (9, 16, 4, (900,), 7, 2),
           (5, 7, 16, (33, 47), 2, 1), (2, 16, 12, (12, 40, 36), 3, 1), (2, 5, 9, (40, 50), 4, 2), (1, 1, 1, (16,), 3, 1)]


@pytest.mark.parametrize("offset", [0, 1], ids=["aligned", "odd"])
@pytest.mark.parametrize("case", SIXTEEN, ids=str)
def test_sixteen_channel_tiles(case, offset):
    """fp32 sums of at most 432 products, and of up to 250000 in the weight gradient (random walk of their roundings)."""
    require_gpu()
    L = ConvLayer(*case, offset=offset)
    assert dd.distdl_debug_conv_kernels(L.plan, offset == 0)[0] == 2
    for run in L.ways():
        L.y.fill_(7.0), L.dx.fill_(5.0)
        for name, got, want in zip(("y", "dx", "dw"), run(), L.exact()):
            assert float((got.double() - want).norm() / want.norm()) < 5e-6, name


@pytest.mark.parametrize("c_in,c_out", [(20, 24), (19, 21), (12, 8)], ids=["split", "gather", "16 x 16"])
@pytest.mark.parametrize("onto", ["w", "dy"])
def test_weight_gradient_in_place(onto, c_in, c_out):
    """dw written onto the weights, or onto a dy that has served: the data gradient reads both as they were."""
    require_gpu()
    L = ConvLayer(2, c_in, c_out, (40, 41), 3, 1)
    want = L.exact()
    L.run()
    L.dw = L.w if onto == "w" else L.dy.view(-1)[:L.w.numel()].view(L.w.shape)
    L.dx.fill_(5.0)
    for name, got, exact in list(zip(("y", "dx", "dw"), L.run(), want))[1:]:
        assert float((got.double() - exact).norm() / exact.norm()) < TOL[F32], name


@pytest.mark.parametrize("c_in,c_out", [(20, 24), (19, 21), (12, 8)], ids=["split", "gather", "16 x 16"])
@pytest.mark.parametrize("pad", [0, 1], ids=["no_halo", "halo"])
def test_a_call_new_to_a_captured_stream_is_refused_and_leaves_the_capture_alone(pad, c_in, c_out):
    require_gpu()
    L = ConvLayer(2, c_in, c_out, (40, 41), 3, 1, p=pad)
    L.run()                                        # (on another stream)
    calls = [lambda: dd.distdl_conv_fwd(L.plan, [L.x], L.w, None, [L.y]),
             lambda: dd.distdl_conv_bwd(L.plan, [L.x], L.w, [L.dy], [L.dx], L.dw, L.db, L.ws)]
    side, graph, mark = torch.cuda.Stream(), torch.cuda.CUDAGraph(), torch.zeros(8, device="cuda")
    torch.cuda.synchronize()
    before = L.x.clone(), L.y.clone(), L.dx.clone()

    def code_of(call):
        try:
            call()
        except dd.DistdlError as error:
            return error.code

    gc.collect()                                   # (plans and graphs of other tests: none may be destroyed during the capture)
    gc.disable()
    try:
        with torch.cuda.graph(graph, stream=side):
            codes = [code_of(call) for call in calls]
            mark.add_(1.0)
    finally:
        gc.enable()
    assert codes == [dd.ERR_INVALID_ARG] * 2
    L.y.fill_(7.0), L.dx.fill_(5.0)
    for _ in range(3):
        graph.replay()
    torch.cuda.synchronize()
    assert bool((mark == 3.0).all()) and bool((L.y == 7.0).all()) and bool((L.dx == 5.0).all())
    L.run()
    assert all(torch.equal(a, b) for a, b in zip(before, (L.x, L.y, L.dx)))


@pytest.mark.parametrize("c_in,c_out", [(20, 24), (19, 21), (28, 3)], ids=["split", "gather", "both"])
@pytest.mark.parametrize("dtype", [F32, BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("pad", [0, 1], ids=["no_halo", "halo"])
def test_weights_ride_in_the_launch_before(pad, dtype, c_in, c_out):
    """The weights are laid out by the halo exchange's launch (none without padding: by one of their own) and by the reduction
    of dw; other weights in the next call are used there."""
    require_gpu()
    L = ConvLayer(2, c_in, c_out, (40, 41), 3, 1, dtype, pad)
    if dtype == BF16 and 4 not in dd.distdl_debug_conv_kernels(L.plan):
        pytest.skip("the bf16 tiles lay out their weights themselves")
    for _ in range(3):
        L.w.copy_(torch.randn_like(L.w))
        dd.distdl_profile_enable(True)
        dd.distdl_profile_report()
        outs = L.run()
        names = set(dd.distdl_profile_report())
        dd.distdl_profile_enable(False)
        if dtype == F32:
            assert ("conv_relayout_w" in names) == (pad == 0)
        for name, got, want in zip(("y", "dx", "dw"), outs, L.exact()):
            assert float((got.double() - want).norm() / want.norm()) < TOL[dtype], name


@pytest.mark.parametrize("P_fo,P_fi", [(1, 9), (9, 1), (9, 10)])
@pytest.mark.parametrize("dtype", [F32, BF16], ids=["f32", "bf16"])
def test_affine_of_more_segments_than_a_product_takes(P_fo, P_fi, dtype):
    """Nine and more blocks to sum over: the direct kernels."""
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(12)
    n_b, n_fi, n_fo = 13, 101, 95
    cut = lambda t, parts, dim: [v.contiguous() for v in torch.tensor_split(t, parts, dim)]
    x, W, b, dy = (torch.randn(sh, generator=g, device="cuda").to(dtype) for sh in ((n_b, n_fi), (n_fo, n_fi), (n_fo,), (n_b, n_fo)))
    xs, dys, bs = cut(x, P_fi, 1), cut(dy, P_fo, 1), cut(b, P_fo, 0)
    Ws = [t for r in cut(W, P_fo, 0) for t in cut(r, P_fi, 1)]
    y, dx, dW, db = ([torch.empty_like(t) for t in ts] for ts in (dys, xs, Ws, bs))
    plan = dd.distdl_affine_plan_create(n_b, n_fi, n_fo, P_fo, P_fi, dtype)
    dd.distdl_profile_enable(True)
    dd.distdl_profile_report()
    dd.distdl_affine_fwd(plan, xs, Ws, bs, y)
    dd.distdl_affine_bwd(plan, xs, Ws, dys, dx, dW, db)
    names = set(dd.distdl_profile_report())
    dd.distdl_profile_enable(False)
    assert ("affine_fwd_direct" in names) == (P_fi > 8) and ("affine_bwd_direct" in names) == (P_fo > 8)
    x, W, b, dy = (t.double() for t in (x, W, b, dy))
    whole = lambda ts: torch.cat([t.double() for t in ts], -1)
    rows = [torch.cat([t.double() for t in dW[i * P_fi:(i + 1) * P_fi]], 1) for i in range(P_fo)]
    for got, want in ((whole(y), x @ W.t() + b), (whole(dx), dy @ W), (torch.cat(rows, 0), dy.t() @ x), (whole(db), dy.sum(0))):
        assert float((got - want).norm() / want.norm()) < TOL[dtype]


@pytest.mark.parametrize("c_in,c_out,cells,k,first", [(44, 12, 1000000, 3, True), (44, 12, 800000, 3, True), (44, 12, 300000, 3, False), (44, 12, 1000000, 1, False),
                                                      (32, 16, 1200000, 3, False)], ids=["large", "141 MB", "small", "one tap", "32-16"])
def test_order_of_the_adjoint(c_in, c_out, cells, k, first):
    """A large dx that a weight gradient of several taps can hide: the data gradient runs first, its weights laid out by a launch of
    their own; elsewhere last, its weights laid out by the reduction of dw.  The same results (sums of at most 132 products, and of a
    million in the weight gradient)."""
    require_gpu()
    L = ConvLayer(1, c_in, c_out, (cells,), k, 1)
    assert dd.distdl_debug_conv_kernels(L.plan)[1:] == (3, 4)
    L.dx.fill_(5.0)
    dd.distdl_conv_fwd(L.plan, [L.x], L.w, None, [L.y])
    dd.distdl_profile_enable(True)
    try:
        dd.distdl_conv_bwd(L.plan, [L.x], L.w, [L.dy], [L.dx], L.dw, L.db, L.ws)
        launches = dd.distdl_profile_report()
    finally:
        dd.distdl_profile_enable(False)
    assert ("conv_relayout_w" in launches) == first
    for name, got, want in zip(("y", "dx", "dw"), (L.y, L.dx[L.bulk], L.dw), L.exact()):
        assert float((got.double() - want).norm() / want.norm()) < TOL[F32], name
