"""Small convolution layers, whose calls run in one launch each way (two where dw is summed over workgroups): against fp64 and
against the general kernels, which the calls without the halo exchange always run."""
import itertools

import numpy as np
import pytest
import torch

import paper_2006_03108_amd as dd
import synthetic_inputs as syn
from oracle import layers
from oracle import primitives as prim
from tests.gpu_util import ConvLayer, assert_close, from_cl, oracle_partition, require_gpu, to_cl, w_to_dev
from tests.test_gpu_conv_kernels import CHOICE, CHOICE_BF16, FEW_ROWS, SIXTEEN
from tests.test_gpu_layers import CONV_ANY, CONV_SPLIT
from tests.test_gpu_split_products import FEW, LAYERS

pytestmark = pytest.mark.gpu
F32, BF16 = torch.float32, torch.bfloat16


def _cfg(n_b, c_in, c_out, shape, P, k, s, p, dil=1):
    each = lambda v: tuple(v) if isinstance(v, (list, tuple)) else (v,) * len(shape)
    return dict(D=len(shape), n_b=n_b, c_in=c_in, c_out=c_out, in_shape=shape, P=each(P), ksize=each(k), stride=each(s), padding=each(p),
                dilation=each(dil), seed=83)


# one tap and many; k that ends within a step of 16 and on it; one to three column tiles; one, two and four waves to a tile; a tile
# for one position; several chunks of weights; strides with classes that no tap reaches, dilations that share a factor with them;
# interior workers (neighbours on both sides of every dimension), padding and halo on one side, uneven parts; all of dw in one
# workgroup and sums over several; channels of 1 ... 164
FUSED = [
    _cfg(1, 1, 1, (64,), 4, 3, 1, 1), _cfg(1, 4, 4, (5,), 2, 1, 1, 0), _cfg(1, 3, 5, (19, 23), (2, 3), (3, 4), (2, 1), (1, 2), (1, 2)),
    _cfg(2, 16, 56, (12, 6), (2, 3), 3, 1, 1), _cfg(2, 5, 33, (9, 11, 10), (3, 3, 2), 3, 1, 1), _cfg(15, 4, 40, (29, 20), 2, 3, 2, 1),
    _cfg(1, 164, 8, (50,), 2, 11, 1, 5), _cfg(2, 8, 12, (13, 14, 15), (3, 1, 3), (2, 3, 1), (2, 3, 1), (1, 1, 0)),
    _cfg(3, 18, 10, (40, 44), (2, 3), 5, 2, 2), _cfg(2, 20, 24, (50,), 3, 7, 4, 3), _cfg(1, 61, 7, (14, 18), (4, 4), 3, 1, 1),
    _cfg(1, 12, 20, (33,), 2, 3, 2, 2, 2), _cfg(2, 8, 8, (4, 4, 4), (2, 2, 2), 2, 1, 1), _cfg(1, 2, 3, (30, 30), (3, 3), 3, 3, 0),
    _cfg(1, 4, 8, (7,), 2, 7, 1, 3), _cfg(6, 4, 4, (40, 41), 1, 3, 1, 1),
]


def _ids(c):
    return f"{c['c_in']}-{c['c_out']}n{'x'.join(map(str, c['in_shape']))}P{'x'.join(map(str, c['P']))}k{c['ksize'][-1]}s{c['stride'][-1]}d{c['dilation'][-1]}"


def _plan(c, dtype):
    return dd.distdl_plan_create(c["D"], c["n_b"], c["c_in"], c["c_out"], c["in_shape"], c["P"], c["ksize"], c["stride"], c["padding"],
                                 c["dilation"], dtype)


class _Layer:
    """offset: every tensor starts that many elements into an allocation"""

    def __init__(self, cfg, dtype, offset=0):
        self.cfg, self.part = cfg, oracle_partition(cfg)
        case = syn.conv_case(cfg, self.part.global_out_shape())
        if dtype == BF16:
            case = {k: (syn.to_bf16_values(v) if isinstance(v, np.ndarray) else v) for k, v in case.items()}
        self.case, self.plan = case, _plan(cfg, dtype)

        def at(t):
            flat = torch.zeros(t.numel() + offset, device="cuda", dtype=dtype)
            flat[offset:] = t.reshape(-1)
            return flat[offset:].view(t.shape)

        self.x = [at(to_cl(b, dtype)) for b in prim.scatter_bulk(case["x"], self.part, fill=np.float32(3.0))]
        self.dy = [at(to_cl(t, dtype)) for t in prim.scatter_out(case["dy"], self.part)]
        self.w, self.b = at(w_to_dev(case["w"]).to(dtype)), at(w_to_dev(case["bias"]).to(dtype))
        self.y, self.dx = ([at(torch.full_like(t, 7.0)) for t in ts] for ts in (self.dy, self.x))
        self.dw, self.db = at(torch.full_like(self.w, 9.0)), at(torch.full_like(self.b, 9.0))
        self.ws = torch.empty(max(dd.distdl_conv_bwd_workspace(self.plan), 16), dtype=torch.uint8, device="cuda")

    def run(self):
        dd.distdl_conv_fwd(self.plan, self.x, self.w, self.b, self.y)
        dd.distdl_conv_bwd(self.plan, self.x, self.w, self.dy, self.dx, self.dw, self.db, self.ws)

    def run_apart(self):
        dd.distdl_halo_fwd(self.plan, self.x)
        dd.distdl_conv_local_fwd(self.plan, self.x, self.w, self.b, self.y)
        dd.distdl_conv_local_bwd(self.plan, self.x, self.w, self.dy, self.dx, self.dw, self.db, self.ws)
        dd.distdl_halo_adj(self.plan, self.dx)

    def outputs(self):
        return [*self.x, *self.y, *self.dx, self.dw, self.db]

    def check(self, tol):
        c, case, part = self.cfg, self.case, self.part
        bufs = prim.scatter_bulk(case["x"].astype(np.float64), part, fill=np.nan)
        y = layers.dist_conv_forward(bufs, case["w"], case["bias"], part, c["stride"], c["dilation"])
        dx, dw, db = layers.dist_conv_adjoint(bufs, case["w"], prim.scatter_out(case["dy"], part), part, c["stride"], c["dilation"], True)
        for w in range(part.n_workers):
            assert np.array_equal(from_cl(self.x[w]), bufs[w].astype(np.float32)), f"x of worker {w}"
            assert_close(from_cl(self.y[w]), y[w], tol, f"y of worker {w}")
            if np.abs(dx[w]).max() > 0:
                assert_close(from_cl(self.dx[w]), dx[w], tol, f"dx of worker {w}")
            else:
                assert not bool(self.dx[w].any())
        assert_close(self.dw.float().cpu().numpy(), dw, tol, "dw")
        assert_close(self.db.float().cpu().numpy(), db, tol, "db")


@pytest.mark.parametrize("offset", [0, 1], ids=["aligned", "odd"])
@pytest.mark.parametrize("dtype", [F32, BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("cfg", FUSED, ids=_ids)
def test_fused_layer(cfg, dtype, offset):
    """fp32: a sum is rounded once (3e-8 of its rms in the mean, 6e-8 at most), in dw also for each of up to a hundred chunks and as
    they are added up: 3e-7; the general kernels' errors, which come on top where the two are compared, are below 5e-7.  bf16: the
    result's rounding, and a value of the other side of it where the sums differ."""
    require_gpu()
    L = _Layer(cfg, dtype, offset)
    fused = dd.distdl_debug_conv_fused(L.plan, offset == 0)
    assert all(fused) if dtype == F32 else any(fused)  # (bf16, 33 and 164 channels: one direction is faster on the gather kernel)
    L.run()
    L.check(3e-7 if dtype == F32 else 2e-2)
    together = [t.clone() for t in L.outputs()]
    L.run()                                          # the same bits again
    assert all(torch.equal(a, b) for a, b in zip(together, L.outputs()))
    L.run_apart()
    for a, b in zip(together, L.outputs()):
        assert float((a.double() - b.double()).norm()) <= (8e-7 if dtype == F32 else 4e-3) * float(b.double().norm())


@pytest.mark.parametrize("cfg", [FUSED[i] for i in (4, 5, 7, 8, 9, 10, 11)], ids=_ids)
def test_fused_layer_with_values_that_are_not_finite(cfg):
    """An infinity in a cell next to a neighbour, and weights that are not finite, which a cell of dx that they do not reach has
    nothing to do with: the numbers, infinities and NaNs of fp64 sums, and of the general kernels (but the 16 x 16 tiles, which make
    NaNs of such weights' products with cells that do not exist)."""
    require_gpu()
    L = _Layer(cfg, F32)
    assert dd.distdl_debug_conv_fused(L.plan) == (True, True) and dd.distdl_debug_conv_kernels(L.plan)[1] != 2
    first, last = (0, 0, *[0] * cfg["D"]), (cfg["c_out"] - 1, 1, *[-1] * cfg["D"])
    L.w[first], L.w[last] = float("inf"), float("nan")
    g = L.plan.query(0)
    L.x[0][(0, *[a + n - 1 for a, n in zip(g["bulk_off"], g["in_size"])], 0)] = float("inf")
    L.dy[-1][(0, *[0] * cfg["D"], 0)] = float("-inf")
    case, part = L.case, L.part
    with np.errstate(invalid="ignore"):
        w = case["w"].astype(np.float64)
        w[first], w[last] = np.inf, np.nan
        whole = case["x"].astype(np.float64)
        whole[(0, 0, *[n - 1 for n in g["in_size"]])] = np.inf
        bufs = prim.scatter_bulk(whole, part, fill=np.nan)
        dy = [t.astype(np.float64) for t in prim.scatter_out(case["dy"], part)]
        dy[-1][(0, 0, *[0] * cfg["D"])] = -np.inf
        y = layers.dist_conv_forward(bufs, w, case["bias"], part, cfg["stride"], cfg["dilation"])
        dx, dw, db = layers.dist_conv_adjoint(bufs, w, dy, part, cfg["stride"], cfg["dilation"], True)
    cl = lambda ts: [torch.from_numpy(np.ascontiguousarray(np.moveaxis(t, 1, -1))).cuda() for t in ts]
    want = [*cl(bufs), *cl(y), *cl(dx), torch.from_numpy(dw).cuda(), torch.from_numpy(db).cuda()]
    L.run()
    together = [t.clone() for t in L.outputs()]
    L.run_apart()
    assert any(bool(torch.isfinite(t).any()) for t in together[-3:]) and not all(bool(torch.isfinite(t).all()) for t in together)
    for a, b, e in zip(together, L.outputs(), want):
        for of in (torch.isnan, torch.isposinf, torch.isneginf):
            assert torch.equal(of(a), of(b)) and torch.equal(of(a), of(e))
        sure = torch.isfinite(b)
        assert float((a[sure].double() - b[sure].double()).norm()) <= 2e-6 * float(b[sure].double().norm())
        assert float((a[sure].double() - e[sure]).norm()) <= 5e-7 * float(e[sure].norm())


def test_fused_calls_from_a_graph_and_on_two_streams():
    require_gpu()
    cfg = _cfg(1, 6, 10, (16, 14), 2, 3, 1, 1)
    L, M = _Layer(cfg, F32), _Layer(dict(cfg, seed=84), F32)
    M.plan = L.plan
    assert dd.distdl_debug_conv_fused(L.plan) == (True, True)
    L.run(), M.run()
    torch.cuda.synchronize()
    want = [[t.clone() for t in v.outputs()] for v in (L, M)]
    one, other, graph = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.stream(one):
        L.run()
        one.synchronize()
        with torch.cuda.graph(graph, stream=one):
            L.run()
    for _ in range(3):
        for t in [*L.y, *L.dx, L.dw, L.db, *M.y, *M.dx, M.dw, M.db]:
            t.fill_(5.0)
        torch.cuda.synchronize()
        for _ in range(10):
            with torch.cuda.stream(one):
                graph.replay()
            with torch.cuda.stream(other):
                M.run()
        torch.cuda.synchronize()
        for v, w in zip((L, M), want):
            assert all(torch.equal(a, b) for a, b in zip(v.outputs(), w))


@pytest.mark.parametrize("onto", ["dx on x", "dx on dy", "db on dw"])
def test_outputs_on_inputs_run_the_general_kernels(onto):
    """What the kernels one after the other make of it, whatever that is: the same as the calls without the halo exchange."""
    require_gpu()
    L = _Layer(_cfg(1, 8, 8, (16, 16), 1, 3, 1, 1), F32)
    assert dd.distdl_debug_conv_fused(L.plan) == (True, True)
    dd.distdl_conv_fwd(L.plan, L.x, L.w, L.b, L.y)
    kept = [t.clone() for t in (*L.x, *L.dy)]
    dw, db = L.dw, L.db

    def adjoint(bwd):
        L.x[0].copy_(kept[0]), L.dy[0].copy_(kept[1]), dw.fill_(0), db.fill_(0)
        dx = L.x[0] if onto == "dx on x" else torch.zeros(2 * L.x[0].numel(), device="cuda")[:L.x[0].numel()].view(L.x[0].shape)
        dy = L.dy[0]
        if onto == "dx on dy":
            dy = dx.view(-1)[:L.dy[0].numel()].view(L.dy[0].shape)
            dy.copy_(L.dy[0])
        out_b = dw.view(-1)[:8] if onto == "db on dw" else db
        dd.distdl_profile_enable(True)
        dd.distdl_profile_report()
        bwd(L.plan, L.x, L.w, [dy], [dx], dw, out_b, L.ws)
        names = set(dd.distdl_profile_report())
        dd.distdl_profile_enable(False)
        assert "conv_bwd_fused" not in names
        return dw.clone()

    first = adjoint(dd.distdl_conv_bwd)
    if onto != "db on dw":                           # (dw is made before dx, or after it, by rules of its own)
        assert torch.equal(first, adjoint(dd.distdl_conv_local_bwd))


@pytest.mark.parametrize("onto", ["w", "bias", "nothing"])
def test_forward_onto_its_weights_runs_the_general_kernels(onto):
    require_gpu()
    L = _Layer(_cfg(1, 8, 8, (16, 16), 1, 3, 1, 1), F32)
    room = torch.empty(8 + L.y[0].numel(), device="cuda")
    y = room[:L.y[0].numel()].view(L.y[0].shape)
    w, b = L.w, L.b
    if onto == "w":
        w = room[-L.w.numel():].view(L.w.shape)   # (its last 8 values lie behind y)
        w.copy_(L.w)
    elif onto == "bias":
        b = room[:8]
        b.copy_(L.b)
    dd.distdl_profile_enable(True)
    dd.distdl_profile_report()
    dd.distdl_conv_fwd(L.plan, L.x, w, b, [y])
    names = set(dd.distdl_profile_report())
    dd.distdl_profile_enable(False)
    assert ("conv_fwd_fused" in names) == (onto == "nothing")


# the layers by which the general kernels are tested elsewhere and that now run in one launch there
SMALL = [(c[1:], dt) for c in CHOICE + FEW_ROWS for dt in (F32,)] + [(c[1:], BF16) for c in CHOICE_BF16 + FEW_ROWS] + \
        [(c, F32) for c in SIXTEEN + LAYERS + FEW]


@pytest.mark.parametrize("offset", [0, 1], ids=["aligned", "odd"])
@pytest.mark.parametrize("case,dtype", SMALL, ids=lambda v: str(v).replace(" ", "") if isinstance(v, tuple) else str(v)[6:])
def test_general_kernels_of_small_layers(case, dtype, offset):
    """The bar of the other parity tests."""
    require_gpu()
    L = ConvLayer(*case, dtype, offset=offset)
    if not any(dd.distdl_debug_conv_fused(L.plan, offset == 0)):
        pytest.skip("runs on the general kernels anyway")
    L.y.fill_(7.0), L.dx.fill_(5.0), L.dw.fill_(9.0)
    dd.distdl_halo_fwd(L.plan, [L.x])
    dd.distdl_conv_local_fwd(L.plan, [L.x], L.w, None, [L.y])
    dd.distdl_conv_local_bwd(L.plan, [L.x], L.w, [L.dy], [L.dx], L.dw, L.db, L.ws)
    for name, got, want in zip(("y", "dx", "dw"), (L.y, L.dx[L.bulk], L.dw), L.exact()):
        assert float((got.double() - want).norm() / want.norm()) < (1e-5 if dtype == F32 else 2e-2), name


@pytest.mark.parametrize("dtype", [F32, BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("cfg", CONV_ANY + CONV_SPLIT, ids=_ids)
def test_general_kernels_of_small_layers_on_several_workers(cfg, dtype):
    require_gpu()
    L = _Layer(dict(cfg, seed=77), dtype)
    if not any(dd.distdl_debug_conv_fused(L.plan)):
        pytest.skip("runs on the general kernels anyway")
    L.run_apart()
    L.check(1e-5 if dtype == F32 else 2e-2)
