"""Small affine layers, whose calls run in one launch each way: against fp64, beside the tiled kernels, which take the larger ones."""
import pytest
import torch

import paper_2006_03108_amd as dd
from oracle import layers
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu

# one of each; tiles of 16 with remainders, K that ends within 4, 16 and 32 and is shared by eight waves, several workers' segments
# of uneven K; rows of whole pieces and of odd lengths; tall, wide, and more workgroups than stay on the chip
SMALL = [(1, 1, 1, 1, 1), (17, 33, 15, 1, 1), (16, 32, 16, 1, 1), (65, 129, 67, 2, 3), (256, 400, 120, 2, 2), (37, 264, 72, 1, 1),
         (200, 1028, 96, 1, 4), (40, 4100, 68, 1, 2), (3, 31, 1037, 2, 1), (48, 192, 264, 3, 1), (601, 260, 388, 2, 2), (1000, 24, 1001, 1, 8)]


@pytest.mark.parametrize("offset", [0, 1], ids=["aligned", "odd"])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("n_b,n_fi,n_fo,P_fo,P_fi", SMALL)
def test_small_affine_against_fp64(n_b, n_fi, n_fo, P_fo, P_fi, dtype, offset):
    """The small kernels sum fp32 tensors in fp64 and round once: each result within 2^-24 of its own.  bf16 results are within
    2^-8 (8 bits), plus sums of up to 4100 products in fp32.  The tiled fp32 kernels: 1e-6 of the 2-norm, as in their own test.  What a plan
    chooses by itself is the one or the other, bit for bit, also from a replayed graph."""
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(n_b * 31 + n_fi)
    new = lambda *shape: torch.randn(int(torch.Size(shape).numel()) + offset, generator=g, device="cuda").to(dtype)[offset:].view(shape)
    size = lambda s: s.stop - s.start
    rows, cols = layers.feature_blocks(n_fo, P_fo), layers.feature_blocks(n_fi, P_fi)
    x, dy = [new(n_b, size(c)) for c in cols], [new(n_b, size(r)) for r in rows]
    W, b = [new(size(r), size(c)) for r in rows for c in cols], [new(size(r)) for r in rows]
    outs = [[new(*t.shape) for t in ts] for ts in (dy, x, W, b)]
    y, dx, dW, db = outs
    plan = dd.distdl_affine_plan_create(n_b, n_fi, n_fo, P_fo, P_fi, dtype)

    def step():
        dd.distdl_affine_fwd(plan, x, W, b, y)
        dd.distdl_affine_bwd(plan, x, W, dy, dx, dW, db)

    def results():
        torch.cuda.synchronize()
        return [[t.clone() for t in ts] for ts in outs]

    got = {}
    for route in (0, 1, -1):
        for t in sum(outs, []):
            t.fill_(7.0)
        dd.distdl_debug_affine_route(plan, route)
        step()
        got[route] = results()
    d = lambda ts: [t.double() for t in ts]
    xd, dyd, Wd, bd = d(x), d(dy), d(W), d(b)
    want = [[sum(xd[j] @ Wd[i * P_fi + j].t() for j in range(P_fi)) + bd[i] for i in range(P_fo)],
            [sum(dyd[i] @ Wd[i * P_fi + j] for i in range(P_fo)) for j in range(P_fi)],
            [dyd[i].t() @ xd[j] for i in range(P_fo) for j in range(P_fi)], [t.sum(0) for t in dyd]]
    for route, tol in ((0, 1e-6), (1, 1.01 * 2.0 ** -24)):
        tol = tol if dtype == torch.float32 else 2.0 ** -8 + 1e-5
        for name, a, e in zip(("y", "dx", "dW", "db"), got[route], want):
            for k, (u, v) in enumerate(zip(a, e)):
                assert float((u.double() - v).norm()) <= tol * float(v.norm()), (route, name, k)
    for a, u, v in zip(*(got[route] for route in (-1, 0, 1))):
        assert all(map(torch.equal, a, u)) or all(map(torch.equal, a, v))

    dd.distdl_debug_affine_route(plan, 1)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        step()
    for scale in (2.0, 0.5):
        for t in x + dy + b:
            t.mul_(scale)
        for t in sum(outs, []):
            t.fill_(7.0)
        torch.cuda.synchronize()
        graph.replay()
        replayed = results()
        step()
        for a, e in zip(replayed, results()):
            assert all(map(torch.equal, a, e))


@pytest.mark.parametrize("route", [-1, 1], ids=["chosen", "small"])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("P_fo,P_fi", [(1, 9), (9, 1), (9, 9)])
def test_more_workers_than_a_block_has_segments(P_fo, P_fi, dtype, route):
    """A block's sum has room for eight segments: of nine workers the small kernels take neither side, and no estimate reads the
    ninth.  fp32 sums of at most 72 products in a chain: 72 roundings of 2^-24; bf16: the result's 2^-8."""
    require_gpu()
    n_b, n_fi, n_fo = 5, 72, 63
    g = torch.Generator(device="cuda").manual_seed(9)
    new = lambda *shape: torch.randn(shape, generator=g, device="cuda").to(dtype)
    size = lambda s: s.stop - s.start
    rows, cols = layers.feature_blocks(n_fo, P_fo), layers.feature_blocks(n_fi, P_fi)
    x, dy = [new(n_b, size(c)) for c in cols], [new(n_b, size(r)) for r in rows]
    W, b = [new(size(r), size(c)) for r in rows for c in cols], [new(size(r)) for r in rows]
    y, dx, dW, db = ([torch.full_like(t, 7.0) for t in ts] for ts in (dy, x, W, b))
    plan = dd.distdl_affine_plan_create(n_b, n_fi, n_fo, P_fo, P_fi, dtype)
    dd.distdl_debug_affine_route(plan, route)
    dd.distdl_profile_enable(True)
    dd.distdl_profile_report()
    dd.distdl_affine_fwd(plan, x, W, b, y)
    dd.distdl_affine_bwd(plan, x, W, dy, dx, dW, db)
    names = set(dd.distdl_profile_report())
    dd.distdl_profile_enable(False)
    assert P_fi <= 8 or "affine_fwd_small" not in names
    assert P_fo <= 8 or "affine_bwd_small" not in names
    xd, dyd = torch.cat(x, 1).double(), torch.cat(dy, 1).double()
    Wd = torch.cat([torch.cat(W[i * P_fi:(i + 1) * P_fi], 1) for i in range(P_fo)]).double()
    got = (torch.cat(y, 1), torch.cat(dx, 1), torch.cat([torch.cat(dW[i * P_fi:(i + 1) * P_fi], 1) for i in range(P_fo)]), torch.cat(db))
    want = (xd @ Wd.t() + torch.cat(b).double(), dyd @ Wd, dyd.t() @ xd, dyd.sum(0))
    for name, u, v in zip(("y", "dx", "dW", "db"), got, want):
        assert float((u.double() - v).norm()) <= (72 * 2.0 ** -24 if dtype == torch.float32 else 2.0 ** -8 + 1e-5) * float(v.norm()), name


@pytest.mark.parametrize("dtype,onto", [(torch.bfloat16, "dW on W"), (torch.bfloat16, "db on W"), (torch.float32, "dW on W"),
                                        (torch.float32, "dx on x"), (torch.float32, "y on x"), (torch.float32, "nothing")],
                         ids=lambda v: v.replace(" ", "_") if isinstance(v, str) else str(v)[6:])
def test_outputs_on_inputs_run_the_tiled_kernels(dtype, onto):
    """The tiled kernels may write behind the last read of what lies below.  bf16: dW and db come after dx, so that either may lie on
    the weights, and the numbers are those of arrays apart."""
    require_gpu()
    n_b, n_f, P = 73, 176, 2
    g = torch.Generator(device="cuda").manual_seed(12)
    new = lambda *shape: torch.randn(shape, generator=g, device="cuda").to(dtype)
    x, dy = [new(n_b, n_f // P) for _ in range(P)], [new(n_b, n_f // P) for _ in range(P)]
    W, b = [new(n_f // P, n_f // P) for _ in range(P * P)], [new(n_f // P) for _ in range(P)]
    y, dx, dW, db = ([torch.full_like(t, 7.0) for t in ts] for ts in (dy, x, W, b))
    plan = dd.distdl_affine_plan_create(n_b, n_f, n_f, P, P, dtype)
    assert dd.distdl_debug_affine_small(plan)[1] and (dtype == torch.bfloat16 or dd.distdl_debug_affine_small(plan)[0])
    dd.distdl_debug_affine_route(plan, 0)
    dd.distdl_affine_bwd(plan, x, W, dy, dx, dW, db)
    want = [t.clone() for t in dx + dW + db]
    dd.distdl_debug_affine_route(plan, -1)
    if onto == "dW on W":
        dW = W
    elif onto == "db on W":
        db = [W[3].view(-1)[i * n_f // P:(i + 1) * n_f // P] for i in range(P)]
    elif onto == "dx on x":
        dx = x
    dd.distdl_profile_enable(True)
    dd.distdl_profile_report()
    dd.distdl_affine_bwd(plan, x, W, dy, dx, dW, db)
    back = set(dd.distdl_profile_report())
    dd.distdl_affine_fwd(plan, x, W, b, x if onto == "y on x" else y)
    ahead = set(dd.distdl_profile_report())
    dd.distdl_profile_enable(False)
    assert ("affine_bwd_small" in back) == (onto in ("nothing", "y on x"))
    assert dtype == torch.bfloat16 or ("affine_fwd_small" in ahead) == (onto != "y on x")
    if dtype == torch.bfloat16:
        assert all(map(torch.equal, dx + dW + db, want))
