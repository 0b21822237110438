"""Host side of the samples in spatial order (no GPU needed): room for every batch size, argument checks, the stream handle."""
import ctypes as C
import random
import types

import pytest

import dg_inputs as di
from paper_2405_04416_amd import binding as B
from paper_2405_04416_amd.step import TrainStep


def _grid(name, log2_T=None):
    g = di.config(name)["grid"]
    return B.dg_grid_desc_init(g["L"], g["F"], log2_T or g["log2_T"], g["n_min"], B.dg_growth_factor(g["n_min"], g["n_max"], g["L"]),
                               di.box_extent(di.config(name)["parts"][0]))


def _need(grid, N):
    order = B.dg_order_desc_init(grid, N)
    return B.dg_hashgrid_encode_bwd_ordered_workspace_bytes(grid, order, N) if order.n_merged else B.dg_hashgrid_encode_bwd_workspace_bytes(grid, N)


@pytest.mark.parametrize("name,n", [("c2_ngp", 13344128), ("c2_ngp", 1 << 24), ("c3_2x2", 6500001), ("c5_share", 1 << 25), ("c4_big", 600000)])
def test_workspace_holds_every_smaller_batch(name, n):
    """The workspace made for up to n samples holds each batch of at most n in one go, whatever number of levels is merged there."""
    step = object.__new__(TrainStep)
    step.occ = None
    grid = _grid(name)
    m = types.SimpleNamespace(grid=grid, mlp=B.dg_mlp_desc(32, 64, 16, 16, 64, 2, 1))
    room, least = step._encode_ws_bytes(m, n), step._order_min(m)
    rng = random.Random(3)
    sizes = [least, n] + [int(n * (0.4 + 0.6 * i / 400)) for i in range(401)] + [rng.randint(1, n) for _ in range(300)]
    for k in sizes:
        want = _need(grid, k) if k >= least else B.dg_hashgrid_encode_bwd_workspace_bytes(grid, k)
        assert want <= room, k


def _counts(grid, order):
    """An ordered call on no samples: its argument checks alone."""
    return B.lib().dg_hashgrid_encode_bwd_ordered_count(C.byref(grid), C.byref(order), None, 0, None, 0, None)


@pytest.mark.parametrize("N", [1, 5000, 1 << 19, 13 << 20, 1 << 26])
def test_order_of_another_grid_is_refused(N):
    """A descriptor serves the grid it was made for (any number of samples) and is refused with a grid whose levels it does not
    fit: the brick sums would be written outside them."""
    names = ["c2_ngp", "c3_2x2", "c4_big", "c5_share"]
    grids = {name: _grid(name) for name in names}
    grids["steep"] = B.dg_grid_desc_init(16, 2, 19, 16, 1.7, [2.0, 2.0, 0.25])
    grids["tall"] = B.dg_grid_desc_init(16, 2, 19, 16, 1.38, [0.25, 2.0, 2.0])
    orders = {name: B.dg_order_desc_init(grid, N) for name, grid in grids.items()}
    refused = 0
    for a, grid in grids.items():
        for b, order in orders.items():
            rc = _counts(grid, order)
            if a == b:
                assert rc == 0, (a, b)
            elif rc != 0:
                refused += 1
                assert B.dg_hashgrid_encode_bwd_ordered_workspace_bytes(grid, order, 1000) == 0
            else:                # accepted: the boxes that this grid's own levels have for these bricks
                assert grid.scale[0][0] / order.n_bricks[0] + 3.02 >= order.box[0][0] or order.box[0][0] == grid.res[0][0] + 1
    assert refused >= 10
    for field in ("per_unit", "box", "box_first"):
        q = B.dg_order_desc_init(grids["c2_ngp"], N)
        if field == "per_unit":
            q.per_unit[1] *= 0.5
        elif field == "box":
            q.box[1][2] += 1
        else:
            q.box_first[2] += 1
        assert _counts(grids["c2_ngp"], q) != 0, field


def test_stream_handle_without_the_raw_getter(monkeypatch):
    """A torch that does not have the getter of raw handles serves the public one."""
    monkeypatch.setattr(B, "_raw_stream", None, raising=False)
    monkeypatch.delattr(B.torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(B.torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=77))
    assert B._stream() == 77


@pytest.mark.parametrize("n_max", [2048, 8192])
@pytest.mark.parametrize("log2_T", range(15, 25))
def test_lines_of_the_order(log2_T, n_max):
    """Where a batch changes to spatial order: at no fewer samples without a backward pass than with one, not yet at sizes where ray order was
    measured to be as fast or faster for views from above, and at sizes where the order was faster by 2 % and more for these and for oblique rays (log2_T, n_max,
    use, samples).  Between the sizes at which the two kinds of rays break even a line is a compromise: T = 2^20 orders 0.84 M samples of a box
    seen from above, 5 % slower there than ray order."""
    faster_in_ray_order = [(18, 2048, "render", 3000000), (19, 2048, "render", 3980000), (19, 2048, "refresh", 1048576), (21, 8192, "step", 602048),
                           (21, 8192, "render", 2070000), (22, 8192, "step", 602560), (22, 8192, "render", 1085000), (17, 2048, "step", 912000),
                           (18, 2048, "step", 1030976), (19, 2048, "step", 891008), (20, 2048, "step", 678528), (21, 2048, "step", 516864),
                           (22, 2048, "step", 379968), (23, 8192, "step", 596448), (24, 8192, "step", 554560), (18, 2048, "render", 3171456),
                           (19, 2048, "render", 4756096), (20, 2048, "render", 1750656), (21, 2048, "render", 675648), (22, 2048, "render", 396224)]
    faster_in_order = [(17, 2048, "step", 1293312), (18, 2048, "step", 1240000), (19, 2048, "step", 1188608), (20, 2048, "step", 1197760),
                       (21, 2048, "step", 795968), (22, 2048, "step", 796608), (21, 8192, "step", 905136), (22, 8192, "step", 768432),
                       (21, 2048, "render", 1193472), (22, 2048, "render", 717824)]
    m = types.SimpleNamespace(grid=B.dg_grid_desc_init(16, 2, log2_T, 16, B.dg_growth_factor(16, n_max, 16), [2.0, 2.0, 0.25]),
                              mlp=B.dg_mlp_desc(32, 64, 16, 16, 64, 2, 1))
    for use in ("step", "render", "refresh"):
        step = object.__new__(TrainStep)
        step.occ, step.ordered = {} if use == "refresh" else None, True
        line = int(step._order_min(m) * step._order_factor(m, use))
        assert step._order_of(m, line - 1, use) is None and step._order_of(m, line, use) is not None
        assert step._order_of(m, step._order_min(m) - 1, use) is None
        for T, finest, what, N in faster_in_ray_order:
            if (T, finest, what) == (log2_T, n_max, use):
                assert step._order_of(m, N, use) is None, N
        for T, finest, what, N in faster_in_order:
            if (T, finest, what) == (log2_T, n_max, use):
                assert step._order_of(m, N, use) is not None, N


@pytest.mark.parametrize("log2_T,occ,use,factor", [(17, True, "step", 1.0), (18, True, "step", 3.0), (24, True, "render", 3.0), (19, True, "refresh", 1.0),
                                                   (20, False, "step", 1.0), (21, False, "step", 1.4), (22, False, "render", 1.4), (22, False, "refresh", 1.0),
                                                   (23, False, "step", 1.0)])
def test_bricks_follow_the_density_of_the_samples(log2_T, occ, use, factor):
    """The bricks are those of the stated multiple of the samples, and the table-gradient workspace that a capacity gets serves every smaller batch."""
    m = types.SimpleNamespace(grid=B.dg_grid_desc_init(16, 2, log2_T, 16, B.dg_growth_factor(16, 2048, 16), [2.0, 2.0, 0.25]),
                              mlp=B.dg_mlp_desc(32, 64, 16, 16, 64, 2, 1))
    step = object.__new__(TrainStep)
    step.occ, step.ordered = {} if occ else None, True
    most = 6000000
    for N in (most, 4000001, 1999999, 1400003):
        if N >= step._order_min(m) * step._order_factor(m, use):
            many = max(N, min(int(N * factor), 1 << 21)) if factor == 1.4 else int(N * factor)
            assert bytes(step._order_of(m, N, use)) == bytes(B.dg_order_desc_init(m.grid, many))
    if use == "step":
        room = step._encode_ws_bytes(m, most)
        for N in range(int(step._order_min(m)), most, 99991):
            assert B.dg_hashgrid_encode_bwd_ordered_workspace_bytes(m.grid, step._order_of(m, N), N) <= room, N


# Bytes that the table-gradient pass has been content with since its queues exist: T = 2^14 .. 2^24, finest level of 2048 and of 8192 cells; samples
# in ray order and in spatial order with the bricks of 2^20 and of 2^25 samples.
SMALLEST_WORKSPACE = {
    2048: [(2759680, 3085568, 3290112), (4898304, 5536768, 6077184), (8819200, 9961216, 11172864), (16037120, 17867776, 20422144),
           (29493504, 32284672, 37524480), (54890240, 50903040, 27959296), (15419136, 18933760, 11974656), (27741440, 31256064, 18802688),
           (50199552, 53713920, 32458752), (91167744, 94682112, 59770880), (159821056, 163335936, 114395136)],
    8192: [(2970624, 3098880, 3303424), (5287424, 5544448, 6084864), (9564928, 10157824, 11369216), (17674496, 18673920, 21228288),
           (33357824, 35028992, 40268800), (62140928, 59350528, 36406784), (18145536, 19295232, 12429824), (33508608, 34658304, 22671872),
           (62795008, 63944448, 43155968), (117419264, 118568704, 84124160), (217825536, 218975232, 166060544)],
}


@pytest.mark.parametrize("n_max", [2048, 8192])
@pytest.mark.parametrize("log2_T", range(14, 25))
def test_smallest_workspace(log2_T, n_max):
    """A workspace in which a call could run in batches stays one: what one tile of 512 samples needs is the least that is accepted."""
    grid = B.dg_grid_desc_init(16, 2, log2_T, 16, B.dg_growth_factor(16, n_max, 16), [2.0, 2.0, 0.25])
    orders = [B.dg_order_desc_init(grid, N) for N in (1 << 20, 1 << 25)]
    least = [B.dg_hashgrid_encode_bwd_workspace_bytes(grid, 512)] + [B.dg_hashgrid_encode_bwd_ordered_workspace_bytes(grid, q, 512) for q in orders]
    for have, most in zip(least, SMALLEST_WORKSPACE[n_max][log2_T - 14]):
        assert 0 < have <= most
