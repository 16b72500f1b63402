"""CPU tests of the library's host side: the C ABI loads and exports every
declared symbol, the planner's geometry agrees with the oracle's independent
planner and with the paper's worked examples, error codes, and the box-task
tables of the one-pass halo kernels -- interpreted here on numpy arrays --
reproduce the oracle's nested halo exchange and its adjoint."""
import os
import random
import re

import numpy as np
import pytest
import torch

import paper_2006_03108_amd as dd
from oracle import geometry as geo
from oracle import primitives as prim

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_declared_symbol_is_exported():
    header = open(os.path.join(ROOT, "include", "distdl.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(distdl_[a-z0-9_]+)\s*\(", header))
    assert len(declared) >= 20
    for name in declared:
        assert hasattr(dd.lib, name), name
    for name in ("distdl_halo_fwd", "distdl_halo_adj", "distdl_bcast_fwd", "distdl_bcast_adj",
                 "distdl_sumreduce_fwd", "distdl_sumreduce_adj", "distdl_conv_fwd", "distdl_conv_bwd",
                 "distdl_affine_fwd", "distdl_affine_bwd"):
        assert name in declared


def _random_setups(count, seed):
    rnd = random.Random(seed)
    out = []
    while len(out) < count:
        D = rnd.randint(1, 3)
        P = [rnd.randint(1, 4) for _ in range(D)]
        k = [rnd.randint(1, 5) for _ in range(D)]
        s = [rnd.randint(1, 3) for _ in range(D)]
        dil = [rnd.randint(1, 2) for _ in range(D)]
        p = [rnd.randint(0, 3) for _ in range(D)]
        n = [rnd.randint(P[d] * 2, P[d] * 7) for d in range(D)]
        out.append((n, P, k, s, p, dil))
    return out


@pytest.mark.parametrize("n,P,k,s,p,dil", _random_setups(60, 1))
def test_planner_agrees_with_oracle_geometry(n, P, k, s, p, dil):
    D = len(n)
    try:
        part = geo.Partition.for_kernel(n, P, k, s, p, dil)
    except geo.EmptyPartition:
        with pytest.raises(dd.DistdlError) as e:
            dd.distdl_plan_create(D, 1, 1, 1, n, P, k, s, p, dil)
        assert e.value.code == dd.ERR_EMPTY_PARTITION
        return
    except geo.HaloTooWide:
        with pytest.raises(dd.DistdlError) as e:
            dd.distdl_plan_create(D, 1, 1, 1, n, P, k, s, p, dil)
        assert e.value.code == dd.ERR_HALO_TOO_WIDE
        return
    plan = dd.distdl_plan_create(D, 2, 3, 4, n, P, k, s, p, dil)
    assert plan.n_workers == part.n_workers
    for w in range(part.n_workers):
        q = plan.query(w)
        for d in range(D):
            g = part.g(w, d)
            assert q["in_start"][d] == g["in_start"] and q["in_size"][d] == g["in_size"]
            assert q["out_start"][d] == g["out_start"] and q["out_size"][d] == g["out_size"]
            assert q["halo"][d] == g["halo"] and q["pad"][d] == g["pad"] and q["extra"][d] == g["extra"]
            assert q["buf_shape"][d] == g["buf"] and q["bulk_off"][d] == g["bulk_off"]
            assert q["conv_origin"][d] == g["origin"]


def test_planner_on_the_papers_pooling_example():
    # App. B.1 fourth example: n = 20, k = 2, s = 2, P = 6
    plan = dd.distdl_plan_create(1, 1, 1, 1, [20], [6], [2], [2], [0], [1])
    got = [(plan.query(w)["halo"][0], plan.query(w)["extra"][0]) for w in range(6)]
    assert got == [((0, 0), (0, 0)), ((0, 0), (0, 0)), ((0, 1), (0, 0)),
                   ((0, 2), (1, 0)), ((0, 1), (2, 0)), ((0, 0), (1, 0))]


def test_error_codes():
    def code(fn):
        with pytest.raises(dd.DistdlError) as e:
            fn()
        return e.value.code
    assert code(lambda: dd.distdl_plan_create(4, 1, 1, 1, [4] * 4, [1] * 4, [1] * 4, [1] * 4, [0] * 4, [1] * 4)) == dd.ERR_INVALID_ARG
    assert code(lambda: dd.distdl_plan_create(1, 0, 1, 1, [4], [1], [1], [1], [0], [1])) == dd.ERR_INVALID_ARG
    assert code(lambda: dd.distdl_plan_create(1, 1, 1, 1, [4], [1], [1], [0], [0], [1])) == dd.ERR_INVALID_ARG
    assert code(lambda: dd.distdl_plan_create(1, 1, 1, 1, [3], [4], [1], [1], [0], [1])) == dd.ERR_EMPTY_PARTITION
    assert code(lambda: dd.distdl_plan_create(1, 1, 1, 1, [8], [4], [7], [1], [3], [1])) == dd.ERR_HALO_TOO_WIDE
    assert code(lambda: dd.distdl_plan_create_explicit(1, 1, 1, [2], [[2, 5]], [[(0, 0), (3, 0)]])) == dd.ERR_HALO_TOO_WIDE
    assert code(lambda: dd.distdl_plan_create_explicit(1, 1, 1, [2], [[0, 5]], [[(0, 0), (0, 0)]])) == dd.ERR_EMPTY_PARTITION
    assert code(lambda: dd.distdl_affine_plan_create(4, 3, 8, 2, 4)) == dd.ERR_EMPTY_PARTITION
    assert code(lambda: dd.distdl_affine_plan_create(0, 3, 8, 1, 1)) == dd.ERR_INVALID_ARG
    assert "worker" in dd.distdl_last_error() or "sizes" in dd.distdl_last_error()
    plan = dd.distdl_plan_create(1, 1, 1, 1, [8], [2], [3], [1], [1], [1])
    with pytest.raises(dd.DistdlError):
        plan.query(2)


def _as3(arr, D):
    """[n_b, n_c, spatial...] -> view with 3 feature dims."""
    return arr.reshape(arr.shape[:2] + (1,) * (3 - D) + arr.shape[2:])


def _box(org, ext):
    return (slice(None), slice(None)) + tuple(slice(o, o + e) for o, e in zip(org, ext))


def _interpret(tasks, bufs, D, adjoint):
    views = [_as3(b, D) for b in bufs]
    for t in tasks:
        dst = views[t["dst"]]
        if not t["srcs"]:
            dst[_box(t["org"], t["ext"])] = 0
        elif not adjoint:
            (sw, sorg), = t["srcs"]
            dst[_box(t["org"], t["ext"])] = views[sw][_box(sorg, t["ext"])]
        else:
            assert [s[0] for s in t["srcs"]] == sorted(s[0] for s in t["srcs"])
            for sw, sorg in t["srcs"]:
                dst[_box(t["org"], t["ext"])] += views[sw][_box(sorg, t["ext"])]
                views[sw][_box(sorg, t["ext"])] = 0


TABLE_SETUPS = [s for s in _random_setups(120, 2)]


@pytest.mark.parametrize("n,P,k,s,p,dil", TABLE_SETUPS[:50] + [
    ([64], [4], [3], [1], [1], [1]), ([12, 12], [2, 2], [3, 3], [1, 1], [1, 1], [1, 1]),
    ([4], [2], [7], [1], [3], [1]),                      # pad and halo on the same side
    ([9, 9], [3, 3], [5, 5], [1, 1], [2, 2], [1, 1]),    # bulk 3 covered from both sides
    ([21, 22, 23], [2, 2, 2], [5, 5, 5], [2, 2, 2], [2, 2, 2], [1, 1, 1])])
def test_task_tables_reproduce_the_oracle_halo_exchange(n, P, k, s, p, dil):
    D = len(n)
    try:
        part = geo.Partition.for_kernel(n, P, k, s, p, dil)
    except ValueError:
        pytest.skip("geometry rejected")
    plan = dd.distdl_plan_create(D, 2, 2, 2, n, P, k, s, p, dil)
    rng = np.random.default_rng(0)
    xg = rng.standard_normal((2, 2) + tuple(n))
    want = prim.halo_exchange(prim.scatter_bulk(xg, part, fill=np.nan), part)
    got = prim.scatter_bulk(xg, part, fill=np.nan)
    _interpret(dd.distdl_debug_tasks(plan, False), got, D, False)
    for a, b in zip(got, want):
        assert np.array_equal(a, b)

    y = [rng.standard_normal(b.shape) for b in want]
    want = prim.halo_exchange_adjoint([t.copy() for t in y], part)
    got = [t.copy() for t in y]
    _interpret(dd.distdl_debug_tasks(plan, True), got, D, True)
    for a, b in zip(got, want):
        np.testing.assert_allclose(a, b, rtol=0, atol=1e-12)


def test_task_tables_cover_every_non_bulk_cell_once():
    part = geo.Partition.for_kernel([10, 11, 9], [2, 3, 2], [5, 3, 4], [1, 1, 2], [2, 1, 1], [1, 1, 1])
    plan = dd.distdl_plan_create(3, 1, 1, 1, [10, 11, 9], [2, 3, 2], [5, 3, 4], [1, 1, 2], [2, 1, 1], [1, 1, 1])
    hits = [np.zeros(part.buf_shape(w), dtype=int) for w in range(part.n_workers)]
    for t in dd.distdl_debug_tasks(plan, False):
        hits[t["dst"]][_box(t["org"], t["ext"])[2:]] += 1
    for w in range(part.n_workers):
        expect = np.ones(part.buf_shape(w), dtype=int)
        expect[part.bulk_slices(w)] = 0
        assert np.array_equal(hits[w], expect)
    # adjoint: every halo cell is read-and-cleared exactly once, every pad cell zeroed once
    hits = [np.zeros(part.buf_shape(w), dtype=int) for w in range(part.n_workers)]
    for t in dd.distdl_debug_tasks(plan, True):
        if not t["srcs"]:
            hits[t["dst"]][_box(t["org"], t["ext"])[2:]] += 1
        for sw, sorg in t["srcs"]:
            hits[sw][_box(sorg, t["ext"])[2:]] += 1
    for w in range(part.n_workers):
        expect = np.ones(part.buf_shape(w), dtype=int)
        expect[part.bulk_slices(w)] = 0
        assert np.array_equal(hits[w], expect)


def test_explicit_plan_matches_app_b2_example():
    plan = dd.distdl_plan_create_explicit(2, 1, 1, [2, 2], [[5, 7], [6, 4]], [[(0, 2), (4, 0)], [(0, 0), (3, 0)]])
    part = geo.Partition.explicit([[5, 7], [6, 4]], [[(0, 2), (4, 0)], [(0, 0), (3, 0)]])
    assert [plan.query(w)["buf_shape"] for w in range(4)] == [list(part.buf_shape(w)) for w in range(4)]
    xg = np.arange(120.0).reshape(1, 1, 12, 10)
    want = prim.halo_exchange(prim.scatter_bulk(xg, part, fill=-1.0), part)
    got = prim.scatter_bulk(xg, part, fill=-1.0)
    _interpret(dd.distdl_debug_tasks(plan, False), got, 2, False)
    for a, b in zip(got, want):
        assert np.array_equal(a, b)


def test_index_decode_division_is_exact():
    rnd = random.Random(3)
    edge = [1, 2, 3, 5, 7, 16, 255, 256, 257, 65535, 65536, 2**31 - 1, 2**31, 2**32 - 1]
    for d in edge + [rnd.randint(1, 2**32 - 1) for _ in range(200)] + [rnd.randint(1, 5000) for _ in range(300)]:
        for n in edge + [0, d - 1, d, d + 1, 2 * d - 1, 2 * d] + [rnd.randint(0, 2**32 - 1) for _ in range(40)]:
            n &= 0xFFFFFFFF
            assert dd.lib.distdl_debug_fastdiv(n, d) == n // d, (n, d)


def test_repartition_plan_blocks_follow_the_balanced_rule_and_errors():
    """The generalized all-to-all's planner (no GPU): its blocks are the oracle's balanced blocks, row-major."""
    from oracle import primitives as prim
    for shape, Ps, Pd in [((3, 10, 9, 8), (1, 2, 3, 2), (3, 1, 2, 4)), ((11,), (4,), (3,)), ((6, 7), (2, 3), (3, 1))]:
        plan = dd.distdl_repart_plan_create(shape, Ps, Pd)
        for side, P in ((0, Ps), (1, Pd)):
            want = [(tuple(s.start for s in sl), tuple(s.stop - s.start for s in sl))
                    for sl in prim.partition_blocks(shape, P)]
            assert plan.blocks(side) == want
    with pytest.raises(dd.DistdlError) as e:
        dd.distdl_repart_plan_create((3, 4), (4, 1), (1, 1))
    assert e.value.code == dd.binding.ERR_EMPTY_PARTITION
    with pytest.raises(dd.DistdlError):
        dd.distdl_repart_plan_create((3, 4, 5, 6, 7), (1,) * 5, (1,) * 5)
    with pytest.raises(dd.DistdlError):
        dd.distdl_repart_plan_create((0, 4), (1, 1), (1, 1))


def test_conv_kernel_family_falls_back_when_no_window_fits():
    """Layers whose staged patch fits no window of the matrix-core correlation (wide dilated kernels with many
    channels) are left to the kernels that take any shape by the planner; they do not fail when the launch is prepared."""
    path = lambda *a, **k: dd.distdl_debug_conv_path(dd.distdl_plan_create(*a, **k))
    # the volumetric configuration and the 2-D one: 32-wide and 16-wide matrix-core tiles
    assert path(3, 1, 32, 32, [64, 64, 64], [2, 2, 2], [5] * 3, [2] * 3, [2] * 3, [1] * 3) == (1, 1, 1)
    assert path(2, 8, 16, 16, [256, 256], [2, 2], [3, 3], [1, 1], [1, 1], [1, 1]) == (2, 2, 2)
    # channel counts that are no multiples of 4: no tiles
    assert path(2, 2, 33, 35, [40, 40], [2, 2], [3, 3], [1, 1], [1, 1], [1, 1])[:2] == (0, 0)
    # k = 3 with dilation 16, k = 7 with dilation 6, 32 channels: the patch of even the narrowest window exceeds
    # the pieces a thread can stage; k = 3 with dilation 3 still fits
    assert path(2, 1, 32, 32, [80, 80], [2, 2], [3, 3], [1, 1], [16, 16], [16, 16])[:2] == (0, 0)
    assert path(2, 1, 32, 32, [90, 90], [2, 2], [7, 7], [1, 1], [18, 18], [6, 6])[:2] == (0, 0)
    assert path(2, 1, 32, 32, [60, 64], [2, 2], [3, 3], [1, 1], [12, 12], [12, 12])[:2] == (1, 1)   # the narrowest window
    assert path(2, 1, 32, 32, [80, 80], [2, 2], [3, 3], [1, 1], [3, 3], [3, 3])[:2] == (1, 1)


def test_conv_kernels_for_shapes_at_the_limits():
    """Which kernels run (0 direct, 1 32-wide tiles, 2 16-wide tiles, 3 split products, 4 gather), where the rules change."""
    run = lambda *a, aligned=True: dd.distdl_debug_conv_kernels(dd.distdl_plan_create(*a), aligned)
    f32, bf16 = torch.float32, torch.bfloat16
    one3 = ([1] * 3,) * 4
    assert run(3, 1, 32, 32, [256] * 3, [4] * 3, [5] * 3, [2] * 3, [2] * 3, [1] * 3, f32) == (3, 3, 3)
    assert run(3, 1, 32, 32, [64] * 3, [2] * 3, [5] * 3, [2] * 3, [2] * 3, [1] * 3, f32, aligned=False) == (4, 4, 4)
    assert run(3, 1, 32, 32, [256] * 3, [4] * 3, [5] * 3, [2] * 3, [2] * 3, [1] * 3, bf16) == (1, 1, 1)
    # a dilation of 16 fits no staged window
    assert run(2, 1, 32, 32, [80, 72], [2, 2], [3, 3], [1, 1], [16, 16], [16, 16], f32)[:2] == (4, 4)
    # 64 stride classes are the last that the gather kernels take, strides of 4 the last of the split ones
    assert run(2, 2, 17, 19, [60, 66], [1, 2], [9, 9], [8, 8], [0, 0], [1, 1], f32) == (4, 4, 4)
    assert run(2, 2, 17, 19, [60, 66], [1, 2], [9, 9], [9, 9], [0, 0], [1, 1], f32) == (0, 0, 0)
    assert run(2, 2, 32, 32, [60, 66], [1, 2], [3, 3], [9, 9], [0, 0], [1, 1], bf16) == (0, 0, 0)
    # tensors of 2 GiB and more: 32-bit offsets no longer reach every element
    assert run(3, 1, 17, 20, [512, 512, 240], *one3[:1], [3] * 3, *one3[1:], f32) == (0, 0, 1)
    # more than 2^32 threads in a launch over all workers, each of whose tensors is small
    many = [3, 1, 17, 17, [1632] * 3, [8] * 3, [3] * 3, [1] * 3, [1] * 3, [1] * 3, f32]
    assert run(*many) == (0, 0, 1)
    many[4] = [1280] * 3
    assert run(*many) == (4, 4, 4)


@pytest.mark.parametrize("plan", [(2, 1, 16640, 32, [9, 9], [1, 1], [5, 5], [4, 4], [2, 2]), (1, 1, 16640, 64, [257], [1], [5], [4], [2]),
                                  (2, 1, 33000, 8, [17, 17], [1, 1], [7, 7], [2, 2], [3, 3]), (1, 1, 8, 65536, [9], [1], [3], [1], [1]),
                                  (1, 1, 65540, 20, [9], [1], [3], [1], [1]), (1, 1, 20, 80000, [9], [1], [1], [4], [0])], ids=str)
def test_columns_of_a_position_fit_16_bits(plan):
    """The split kernels for few channels hold the bounds of a position's columns in 16 bits each: a launch of more columns is
    one of the general form, with one cell to a position and no products that two taps share."""
    p = dd.distdl_plan_create(*plan, [1] * plan[0])
    for backward in (False, True):
        _, fold, columns, pairs, _ = dd.distdl_debug_conv_split(p, backward)
        assert columns <= 0xffff or (fold == 1 and pairs == 0)


def test_kernels_of_wide_layers_of_16_channels():
    """16 -> 16 channels, 3 x 3: 16 x 16 tiles (2) forward and in the data gradient, on one worker and on four."""
    for n in (192, 256, 320):
        for P in ([1, 1], [2, 2]):
            assert dd.distdl_debug_conv_kernels(dd.distdl_plan_create(2, 8, 16, 16, [n, n], P, [3, 3], [1, 1], [1, 1], [1, 1]))[:2] == (2, 2)


@pytest.mark.parametrize("plan,kernel", [((2, 8, 4, 4, [660, 860], [1, 2], [5, 5], [1, 1], [0, 0]), 3),
                                         ((2, 1, 28, 60, [794, 1047], [1, 2], [2, 2], [1, 1], [1, 1], [2, 2]), 3),
                                         ((2, 8, 16, 16, [256, 256], [2, 2], [3, 3], [1, 1], [1, 1]), 2),
                                         ((1, 2, 16, 4, [4000], [1], [3], [1], [1]), 4),
                                         ((3, 7, 56, 36, [66, 57, 74], [2, 2, 2], [1, 1, 1], [1, 1, 1], [0, 0, 0]), 4),
                                         ((3, 7, 40, 40, [33, 60, 52], [2, 2, 2], [1, 1, 1], [1, 1, 1], [0, 0, 0]), 4),
                                         ((2, 9, 4, 40, [235, 43], [1, 2], [3, 3], [1, 1], [0, 0]), 4)], ids=str)
def test_weight_gradient_kernel_of_layers_far_from_the_lines(plan, kernel):
    """Layers where one kernel of the weight gradient (2 16 x 16 tiles, 3 split products, 4 gather) is well ahead of the others."""
    plan = plan if len(plan) == 10 else (*plan, [1] * plan[0])
    assert dd.distdl_debug_conv_kernels(dd.distdl_plan_create(*plan))[2] == kernel


@pytest.mark.parametrize("plan,kernel", [((1, 8, 8, 11, [30], [2], [7], [2], [0]), 4), ((2, 2, 8, 9, [22, 134], [1, 1], [7, 7], [1, 2], [3, 3]), 4),
                                         ((2, 15, 5, 10, [84, 79], [1, 1], [5, 5], [2, 2], [2, 2]), 4),
                                         ((1, 9, 8, 16, [33496], [1], [7], [2], [3]), 3), ((1, 10, 1, 4, [36990], [1], [1], [2], [0]), 3)], ids=str)
def test_data_gradient_in_classes_of_a_stride(plan, kernel):
    """One launch of the gather kernel (4) or of folded cells (3) in place of one of the 16 x 16 tiles for each class."""
    assert dd.distdl_debug_conv_kernels(dd.distdl_plan_create(*plan, [1] * plan[0]))[1] == kernel


@pytest.mark.parametrize("plan,kernels", [((2, 2, 32, 32, [60, 64], [1, 1], [3, 3], [1, 1], [1, 1]), (4, 4, 4)),
                                          ((2, 5, 24, 32, [35, 382], [2, 1], [3, 3], [1, 1], [0, 0]), (4, 1, 4)),
                                          ((2, 6, 24, 24, [10, 288], [1, 1], [5, 5], [2, 2], [2, 2]), (1, 4, 4)),
                                          ((2, 7, 24, 48, [16, 31], [1, 1], [5, 5], [1, 1], [0, 0]), (1, 1, 4)),
                                          ((2, 6, 8, 32, [77, 486], [1, 1], [3, 3], [2, 2], [0, 0]), (4, 4, 4)),
                                          ((3, 3, 48, 8, [55, 30, 33], [1, 2, 1], [3, 3, 3], [1, 1, 1], [1, 1, 1]), (1, 1, 1))], ids=str)
def test_bf16_kernels_of_layers_that_the_other_choice_slows_down(plan, kernels):
    """bf16 layers that take 1.1 to 2.4 times as long with the weight gradient on the other kernel (1 tiles, 4 gather), which the other
    two directions may follow."""
    assert dd.distdl_debug_conv_kernels(dd.distdl_plan_create(*plan, [1] * plan[0], torch.bfloat16)) == kernels


def test_bf16_weight_gradient_of_wide_rows_and_several_planes():
    """1404 rows, 3 columns: tiles of 256 rows (73 us, of 64 rows 93)."""
    plan = dd.distdl_plan_create(3, 8, 52, 3, [77, 50, 22], [1] * 3, [3] * 3, [2] * 3, [1] * 3, [1] * 3, torch.bfloat16)
    assert dd.distdl_debug_conv_wgrad_rows(plan) == 256


def test_cells_under_a_dilation_are_folded_only_where_it_pays():
    """Forward passes of three dimensions, dilation 2: in the general form (one cell to a position) where folding took 1.2 to 1.3 times as
    long, folded where it takes 0.9."""
    plan = lambda n_b, c_in, c_out, n: dd.distdl_plan_create(3, n_b, c_in, c_out, n, [1] * 3, [5] * 3, [1] * 3, [4] * 3, [2] * 3)
    assert dd.distdl_debug_conv_split(plan(4, 48, 8, [30, 41, 36]))[1] == 1
    assert dd.distdl_debug_conv_split(plan(4, 32, 10, [29, 29, 38]))[1] == 1
    assert dd.distdl_debug_conv_split(plan(8, 56, 3, [27, 32, 55]))[1] > 1


def test_search_of_launch_shapes_is_short():
    """A plan is searched in its first call: of the hundreds of thousand windows of its folds, classes and M-tiles a few are tried."""
    for plan, most in (((2, 6, 4, 4, [528, 776], [1, 1], [5, 5], [1, 1], [2, 2]), 2500), ((1, 2, 4, 2, [1170], [1], [7], [1], [3]), 2500),
                       ((2, 8, 16, 16, [256, 256], [2, 2], [3, 3], [1, 1], [1, 1]), 400), ((2, 8, 3, 32, [224, 224], [2, 2], [7, 7], [2, 2], [3, 3]), 800),
                       ((3, 1, 4, 4, [300] * 3, [2] * 3, [5] * 3, [2] * 3, [2] * 3), 3000)):
        p = dd.distdl_plan_create(*plan, [1] * plan[0])
        dd.distdl_debug_conv_kernels(p)
        assert dd.distdl_debug_conv_split(p)[4] <= most, plan


def test_table_cache_policy_never_rewrites_a_block_another_reader_may_hold():
    """The device-table cache (pointer arrays, GEMM descriptors), run without a device: eight blocks per stream with
    least-recently-used replacement, no replacement across streams, blocks selected during capture pinned for good,
    unknown tables refused during capture, and an error instead of an eviction when nothing may be reused."""
    pol = dd.distdl_debug_slot_policy
    # steady state: a repeated table reuses its block
    assert pol([0, 0, 0, 0], [7, 8, 7, 8], [0] * 4) == [0, 1, 0, 1]
    # the ninth distinct table on a stream replaces that stream's least recently used block
    seq = list(range(1, 10))
    assert pol([0] * 9, seq, [0] * 9) == [0, 1, 2, 3, 4, 5, 6, 7, 0]
    assert pol([0] * 10, [1, 2, 3, 4, 5, 6, 7, 8, 1, 9], [0] * 10)[-1] == 1      # table 1 was touched again: 2 goes
    # another stream never takes over a block: the same table on stream 1 gets a block of its own, and stream 1's
    # ninth table replaces one of ITS blocks
    got = pol([0, 1] + [1] * 8, [5, 5] + list(range(10, 18)), [0] * 10)
    assert got[0] == 0 and got[1] == 1 and got[-1] == 1 and 0 not in got[1:]
    # a table first seen during capture is refused (its copy would read host memory at replay)
    assert pol([0, 0], [1, 2], [0, 1]) == [0, dd.ERR_INVALID_ARG]
    # a block selected during capture is pinned: eight more tables on the stream leave it alone ...
    got = pol([0] * 11, [1, 1] + list(range(2, 11)), [0, 1] + [0] * 9)
    assert got[1] == 0 and 0 not in got[2:]
    # ... and the recorded table is still found afterwards
    assert pol([0] * 12, [1, 1] + list(range(2, 11)) + [1], [0, 1] + [0] * 10)[-1] == 0
    # 64 blocks, all pinned by captures: the next new table fails with NOMEM instead of evicting one
    streams, tables, cap = [], [], []
    for t in range(64):
        streams += [0, 0]
        tables += [100 + t, 100 + t]
        cap += [0, 1]
    got = pol(streams + [0], tables + [999], cap + [0])
    assert sorted(set(got[:-1])) == list(range(64)) and got[-1] == dd.ERR_NOMEM


@pytest.mark.parametrize("missing", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_stream_handle_without_torchs_private_functions(monkeypatch, missing):
    """A torch build that lacks one of them: the handle comes from the stream object."""
    from paper_2006_03108_amd import binding

    class Stream:
        cuda_stream = 7

    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: Stream)
    for name, fn in (("_cuda_getCurrentRawStream", lambda device: 5 + device), ("_cuda_getDevice", lambda: 1)):
        monkeypatch.setattr(torch._C, name, fn, raising=False)
    assert binding._stream() == 6
    monkeypatch.delattr(torch._C, missing)
    assert binding._stream() == 7


def test_choice_of_the_fused_kernels_is_that_of_the_call():
    """What the launches apart are estimated at depends on the alignment of the weights, too (bf16: tiles or the gather kernel): a
    plan answers for either whatever it was asked before."""
    def plan():
        return dd.distdl_plan_create(3, 1, 20, 4, [7, 7, 5], [2, 2, 1], [5] * 3, [2] * 3, [2] * 3, [1] * 3, torch.bfloat16)
    first, second = plan(), plan()
    answers = {aligned: dd.distdl_debug_conv_fused(first, aligned) for aligned in (1, 2)}
    assert answers[1] != answers[2]
    assert {aligned: dd.distdl_debug_conv_fused(second, aligned) for aligned in (2, 1)} == answers


@pytest.mark.parametrize("n_b,c_in,c_out,n,P,k,p,dil,dtype", [
    (13, 5, 1, (7, 9, 6), (1, 3, 2), 3, 0, 2, torch.float32), (10, 16, 36, (14, 12, 15), (2, 3, 2), 2, 0, 1, torch.float32),
    (4, 4, 4, (156, 120), (1, 2), 2, 1, 1, torch.bfloat16), (10, 8, 4, (7710,), (2,), 5, 2, 2, torch.bfloat16)])
def test_no_margin_leaves_an_adjoint_to_launches_that_take_half_as_long_again(n_b, c_in, c_out, n, P, k, p, dil, dtype):
    """Measured at 30.8 us apart and 17.1 together, 48.5 / 32.6, 26.3 / 16.5, 27.1 / 18.2."""
    D = len(n)
    plan = dd.distdl_plan_create(D, n_b, c_in, c_out, n, P, (k,) * D, (1,) * D, (p,) * D, (dil,) * D, dtype)
    assert dd.distdl_debug_conv_fused(plan)[1]


@pytest.mark.parametrize("n_b,c_in,c_out,n,P,k,dil", [
    (3, 12, 4, (8, 6, 6), (3, 3, 3), 1, 1), (2, 2, 9, (19, 14), (4, 4), 1, 2), (1, 4, 4, (28, 31), (4, 2), 1, 2)])
def test_adjoints_without_an_exchange_have_a_launch_less_to_save(n_b, c_in, c_out, n, P, k, dil):
    """No halos, no H*: measured at 19.6 us apart and 25.9 together, 17.0 / 22.0, 14.9 / 18.7."""
    D = len(n)
    assert not dd.distdl_debug_conv_fused(dd.distdl_plan_create(D, n_b, c_in, c_out, n, P, (k,) * D, (1,) * D, (0,) * D, (dil,) * D))[1]


@pytest.mark.parametrize("n_b,n_fi,n_fo,P_fo,P_fi,by_alignment", [
    (144, 2500, 1384, 3, 1, {2: False, 4: True, 16: True}),  # rows of whole words, none of whole 16-byte pieces
    (115, 552, 1485, 1, 3, {2: False, 4: True, 16: False}),  # whole pieces: the bf16 tiles
])
def test_choice_of_the_small_affine_kernels_is_that_of_the_call(n_b, n_fi, n_fo, P_fo, P_fi, by_alignment):
    """bf16 rows that do not start on a word move value by value, which the forward estimate knows: a plan answers for either
    whatever it was asked before.  (Layers near the line, where the answers differ.)"""
    for order in (list(by_alignment), list(by_alignment)[::-1]):
        plan = dd.distdl_affine_plan_create(n_b, n_fi, n_fo, P_fo, P_fi, torch.bfloat16)
        assert {align: dd.distdl_debug_affine_small(plan, align)[0] for align in order} == by_alignment


@pytest.mark.parametrize("n_b,n_fi,n_fo,P_fo,P_fi", [(38, 2656, 1776, 4, 3), (138, 1488, 2512, 3, 3), (30, 3248, 7040, 2, 2), (22, 1744, 6352, 2, 1)])
def test_small_affine_layers_of_two_workgroups_a_compute_unit(n_b, n_fi, n_fo, P_fo, P_fi):
    """256 to 512 workgroups forward are two rounds but for a quarter: tiled 20.9 us against 29.1 (138 x 1488 -> 2512), 29.9 / 38.8, 19.4 / 22.6."""
    assert not dd.distdl_debug_affine_small(dd.distdl_affine_plan_create(n_b, n_fi, n_fo, P_fo, P_fi, torch.float32))[0]


@pytest.mark.parametrize("n_b,n_fi,n_fo,P_fo,P_fi", [(98, 64, 160, 1, 3), (13, 53, 253, 2, 3), (3, 30, 11, 1, 1)])
def test_the_least_that_a_call_costs_the_host_keeps_no_small_affine_layer_from_one_launch(n_b, n_fi, n_fo, P_fo, P_fi):
    """bf16 of odd rows, forward: where both estimates are little more than the host's time, the launch of small layers is the faster one."""
    assert dd.distdl_debug_affine_small(dd.distdl_affine_plan_create(n_b, n_fi, n_fo, P_fo, P_fi, torch.bfloat16))[0]


@pytest.mark.parametrize("seed", range(40))
def test_overlap_of_a_calls_arrays(seed):
    """Against every pair, for arrays in order, in reverse, interleaved, at random, with and without one that touches another."""
    rng = random.Random(seed)
    for _ in range(40):
        n_groups, n = rng.randint(1, 8), rng.choice([1, 1, 2, 5, 17])
        kinds = [rng.random() < 0.5 for _ in range(n_groups)]
        slots = [(g, i) for g in range(n_groups) for i in range(n)]
        order = rng.choice(["blocks", "interleaved", "random"])
        if order == "interleaved":
            slots.sort(key=lambda s: (s[1], s[0]))
        elif order == "random":
            rng.shuffle(slots)
        at, place = 4096, {}
        for s in slots:
            size = rng.choice([0, 2, 64, 1000])
            place[s] = (at, size)
            at += size + rng.choice([0, 0, 2, 512])
        for _ in range(rng.choice([0, 0, 1, 2])):                     # an array moved onto another one's place
            a, b = rng.choice(slots), rng.choice(slots)
            place[a] = (place[b][0] + rng.choice([-3, 0, 1, place[b][1]]), place[a][1])
        if rng.random() < 0.2:
            place[rng.choice(slots)] = (0, 64)                        # no array
        groups = [(kinds[g], [place[g, i] for i in range(n)]) for g in range(n_groups)]
        for k in range(n_groups):
            if rng.random() < 0.3:
                groups[k][1].reverse()
        arrays = [(a, a + b, out) for out, g in groups for a, b in g if a and b]
        want = any(p[0] < q[1] and q[0] < p[1] and (p[2] or q[2]) for i, p in enumerate(arrays) for q in arrays[:i])
        assert dd.distdl_debug_overlap(groups) == want


def test_overlap_of_many_workers_arrays():
    """A thousand workers' arrays, allocated worker by worker or in any order: sixteen times as many take some sixteen times as long
    (sorted: 16 * 12 / 8 = 24), where comparing each with each took 256 times as long."""
    import ctypes as C
    import time

    def least(n, shuffled):
        places = list(range(3 * n))
        if shuffled:
            random.Random(1).shuffle(places)
        first = [4096 * (1 + places[3 * i + g]) for g in range(3) for i in range(n)]
        args = ((C.c_uint64 * (3 * n))(*first), (C.c_uint64 * (3 * n))(*[4096] * (3 * n)), (C.c_int32 * 3)(n, n, n), (C.c_int32 * 3)(0, 0, 1), 3)
        best = float("inf")
        for _ in range(50):
            t = time.perf_counter()
            assert dd.lib.distdl_debug_overlap(*args) == 0
            best = min(best, time.perf_counter() - t)
        return best

    for shuffled in (False, True):
        assert least(1024, shuffled) < 80 * least(64, shuffled)


def test_choice_of_the_fused_kernels_makes_no_tables():
    """A thousand workers, a stride of 4 x 4 x 4: 65536 records of 176 bytes and more, 11.5 MB a plan, which a layer that goes another
    way has no use for."""
    def resident():
        with open("/proc/self/statm") as f:
            return int(f.read().split()[1]) * os.sysconf("SC_PAGE_SIZE")
    new = lambda: dd.distdl_plan_create(3, 1, 8, 8, [64, 64, 128], [8, 8, 16], [4] * 3, [4] * 3, [0] * 3, [1] * 3)
    assert dd.distdl_debug_conv_fused(new()) == (False, False)  # (what the first use of anything takes)
    plans = [new() for _ in range(6)]
    before = resident()
    assert all(dd.distdl_debug_conv_fused(p) == (False, False) for p in plans)
    assert resident() - before < 6 * 5e6
