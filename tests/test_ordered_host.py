"""Host side of the samples in spatial order (no GPU needed): room for every batch size, argument checks, the stream handle."""
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
