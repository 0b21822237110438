"""Samples in spatial order: the sort, the encode into rows, the table gradient with merged levels, and the training step
that uses them, at the sizes where they can go wrong -- one sample, one more than a wavefront or a workgroup takes, a brick
that holds several pieces, samples on the box's faces and outside it."""
import numpy as np
import pytest
import torch

import dg_inputs as di
import oracle
from gpu_util import DEV, TOL_F16, dev, have_gpu, host, rel_err
from paper_2405_04416_amd import binding as B
from paper_2405_04416_amd.step import TrainStep

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not have_gpu(), reason="needs a GPU")]

GRIDS = {"cached": dict(log2_T=14, n_max=256, extent=[2.0, 2.0, 0.25]), "large": dict(log2_T=20, n_max=2048, extent=[1.0, 0.7, 0.3])}
FLAVOURS = ("points", "one_spot", "faces")
SIZES = (1, 63, 1023, 1025, 4097, 20011)


def _grids(key):
    q = GRIDS[key]
    growth = B.dg_growth_factor(16, q["n_max"], 16)
    return B.dg_grid_desc_init(16, 2, q["log2_T"], 16, growth, q["extent"]), oracle.grid_init(16, 2, q["log2_T"], 16, growth, q["extent"])


def _coords(N, flavour):
    u = di.make_unit_coords(N, seed=31)
    if flavour == "one_spot":                       # everything in one brick: several pieces of it where N > 4096
        u = (0.37 + 1e-3 * u).astype(np.float32)
    if flavour == "faces":                          # corners, faces, and coordinates beyond the box (clamped by the encode)
        special = np.asarray([[0, 0, 0], [1, 1, 1], [-0.3, 0.5, 2.0], [1, 0, 0.5], [0.99999994, 0.5, 0.0], [0.5, 1.0, 0.25]], np.float32)
        n = min(N, len(special))
        u[:n] = special[:n]
    return u


def _sorted(grid, u, N):
    order = B.dg_order_desc_init(grid, N)
    ordered = torch.full((N, 4), float("nan"), device=DEV)
    pieces = torch.full((B.dg_order_pieces_words(order, N),), -1, dtype=torch.int32, device=DEV)
    ws = torch.full((B.dg_order_workspace_bytes(order) // 4,), -7, dtype=torch.int32, device=DEV)
    B.dg_order_samples(order, dev(u), N, ordered, pieces, ws)
    return order, ordered, pieces


def _mixed(g, M):
    """Gradient [N, 32] as the ordered backward pass reads it: rows of the first M levels, then planes."""
    return np.concatenate([np.ascontiguousarray(g[:, :2 * M]).ravel(), np.ascontiguousarray(g[:, 2 * M:].reshape(len(g), 16 - M, 2).transpose(1, 0, 2)).ravel()])


@pytest.mark.parametrize("flavour", FLAVOURS)
@pytest.mark.parametrize("N", SIZES)
@pytest.mark.parametrize("key", list(GRIDS))
def test_ordered_encode(key, N, flavour):
    print("[case] ordered", key, N, flavour, flush=True)
    grid, ref_grid = _grids(key)
    u = _coords(N, flavour)
    order, ordered, pieces = _sorted(grid, u, N)
    M = order.n_merged
    assert M >= 2 and order.total >= 1

    # the sorted list is a permutation that carries the coordinates along; the pieces pave it, at most 4096 samples each
    got = host(ordered)
    index = got[:, 3].copy().view(np.uint32)
    np.testing.assert_array_equal(np.sort(index), np.arange(N))
    np.testing.assert_array_equal(got[:, :3].view(np.uint32), u[index].view(np.uint32))
    words = host(pieces).view(np.uint32).reshape(-1, 2)
    n_pieces = int(words[0, 0])
    begins = words[1:2 + n_pieces, 1].astype(np.int64)
    assert begins[0] == 0 and begins[-1] == N and np.all(np.diff(begins) > 0) and np.all(np.diff(begins) <= 4096)

    # forward: rows in the original order; fp16 of an fp32 sum (bound as in the plain encode's test)
    table = di.make_table(ref_grid.n_entries, 2, 1.0, seed=32)
    rows = torch.full((N, 32), float("nan"), dtype=torch.float16, device=DEV)
    B.dg_hashgrid_encode_fwd_ordered(grid, dev(table), ordered, N, rows)
    ref = oracle.encode_fwd(ref_grid, table, u)
    bound = oracle.encode_fwd(ref_grid, table, u, abs_terms=True)
    assert np.all(np.abs(host(rows).astype(np.float64) - ref) <= 2.0 ** -11 * np.abs(ref) + 1e-5 * bound + 6e-8)

    # backward, called twice ("+="); rows of the merged levels, then planes
    g = (np.random.default_rng(33).standard_normal((N, 32)) * 1e-3).astype(np.float32)
    g[::7] = 0.0
    mixed = np.concatenate([np.ascontiguousarray(g[:, :2 * M]).ravel(), np.ascontiguousarray(g[:, 2 * M:].reshape(N, 16 - M, 2).transpose(1, 0, 2)).ravel()])
    ud, gd = dev(u), dev(mixed)
    dtable = torch.zeros(ref_grid.n_entries, 2, device=DEV)
    ws = torch.zeros(B.dg_hashgrid_encode_bwd_ordered_workspace_bytes(grid, order, N) // 4 + 64, device=DEV)
    largest = gd.abs().max().reshape(1).view(torch.int32)
    B.dg_hashgrid_encode_bwd_ordered(grid, order, ordered, pieces, ud, gd, largest, N, dtable, ws)
    B.dg_hashgrid_encode_bwd_ordered_count(grid, order, ud, N, ws)
    B.dg_hashgrid_encode_bwd_ordered(grid, order, ordered, pieces, ud, gd, largest, N, dtable, ws, counted=True)
    want = 2.0 * oracle.encode_bwd(ref_grid, u, g.astype(np.float64))
    scale = 2.0 * oracle.encode_bwd(ref_grid, u, np.abs(g).astype(np.float64))          # sum of the contributions' magnitudes
    have = host(dtable).astype(np.float64)
    for l in range(16):
        sl = slice(ref_grid.first[l], ref_grid.first[l + 1])
        if l < M:
            # a run adds up to 2 x 64 contributions in fp32, each of them four fp32 roundings deep; the rest is exact up to its
            # quantum (2^-37 of the largest gradient, at most one half per contribution) and a handful of fp32 adds into the
            # table: (128 + 8) x 2^-24 of the magnitudes = 8.1e-6
            quantum = 2.0 ** -37 * float(np.abs(g).max()) * (2 * N)
            assert np.all(np.abs(have[sl] - want[sl]) <= 1e-5 * scale[sl] + quantum), l
        else:
            assert rel_err(have[sl], want[sl]) <= TOL_F16, l                             # the binned pass, with its own bar
    assert np.all(have[want == 0] == 0)


@pytest.mark.parametrize("key", list(GRIDS))
def test_ordered_backward_in_batches(key):
    """A workspace that holds half of the samples: the unmerged levels go through it in batches, the merged ones do not use it."""
    print("[case] ordered in batches", key, flush=True)
    grid, ref_grid = _grids(key)
    N = 20011
    u = _coords(N, "points")
    order, ordered, pieces = _sorted(grid, u, N)
    M = order.n_merged
    need = B.dg_hashgrid_encode_bwd_ordered_workspace_bytes(grid, order, N // 2 + 512)
    assert need < B.dg_hashgrid_encode_bwd_ordered_workspace_bytes(grid, order, N)
    g = (np.random.default_rng(34).standard_normal((N, 32)) * 1e-3).astype(np.float32)
    mixed = np.concatenate([np.ascontiguousarray(g[:, :2 * M]).ravel(), np.ascontiguousarray(g[:, 2 * M:].reshape(N, 16 - M, 2).transpose(1, 0, 2)).ravel()])
    gd = dev(mixed)
    dtable, ws = torch.zeros(ref_grid.n_entries, 2, device=DEV), torch.zeros(need // 4, device=DEV)
    B.dg_hashgrid_encode_bwd_ordered(grid, order, ordered, pieces, dev(u), gd, gd.abs().max().reshape(1).view(torch.int32), N, dtable, ws)
    want, have = oracle.encode_bwd(ref_grid, u, g.astype(np.float64)), host(dtable).astype(np.float64)
    for l in range(16):
        sl = slice(ref_grid.first[l], ref_grid.first[l + 1])
        assert rel_err(have[sl], want[sl]) <= TOL_F16, l


@pytest.mark.parametrize("N", [1025, 20011])
@pytest.mark.parametrize("key", list(GRIDS))
def test_small_gradients_beside_a_large_one(key, N):
    """Levels whose tables together have at most 8192 entries are summed in floating point from end to end: gradients 2^-44
    times as large as the largest keep their fp32 precision there."""
    print("[case] small gradients", key, N, flush=True)
    grid, ref_grid = _grids(key)
    u = np.minimum(_coords(N, "points"), np.float32(0.7))
    u[0] = 0.999                                     # the large one has its cells for itself
    g = (np.random.default_rng(35).standard_normal((N, 32)) * 2.0 ** -44).astype(np.float32)
    g[0] = 1.0
    order, ordered, pieces = _sorted(grid, u, N)
    M = order.n_merged
    gd = dev(_mixed(g, M))
    dtable = torch.zeros(ref_grid.n_entries, 2, device=DEV)
    ws = torch.zeros(B.dg_hashgrid_encode_bwd_ordered_workspace_bytes(grid, order, N) // 4 + 64, device=DEV)
    B.dg_hashgrid_encode_bwd_ordered(grid, order, ordered, pieces, dev(u), gd, gd.abs().max().reshape(1).view(torch.int32), N, dtable, ws)
    want = oracle.encode_bwd(ref_grid, u, g.astype(np.float64))
    scale = oracle.encode_bwd(ref_grid, u, np.abs(g).astype(np.float64))
    have = host(dtable).astype(np.float64)
    coarse = [l for l in range(16) if ref_grid.first[l + 1] <= 8192]
    assert len(coarse) >= 2
    for l in coarse:
        sl = slice(ref_grid.first[l], ref_grid.first[l + 1])
        # a contribution is four fp32 roundings deep and goes through at most seven adds in a run; then fp64, rounded once
        assert np.all(np.abs(have[sl] - want[sl]) <= 12 * 2.0 ** -24 * scale[sl]), l


# the cuts that batches of some millions of samples get: several bricks along every axis, up to twelve merged levels, more
# bricks than 64 KB of LDS count
CUTS = {"flat": dict(log2_T=19, n_max=2048, extent=[2.0, 2.0, 0.25], made_for=13300000, bricks=[53, 53, 6], n_merged=12),
        "upright": dict(log2_T=17, n_max=2048, extent=[0.25, 2.0, 2.0], made_for=20 << 20, bricks=[6, 53, 53], n_merged=12),
        "cube": dict(log2_T=16, n_max=1024, extent=[1.0, 1.0, 1.0], made_for=1 << 26, bricks=[31, 31, 31], n_merged=10),
        "fine": dict(log2_T=16, n_max=8192, extent=[2.0, 2.0, 0.25], made_for=1 << 25, bricks=[60, 60, 7], n_merged=10)}


def _beside_faces(order, N, rng):
    """Coordinates of which three quarters lie on a brick's face along some axis, exactly or up to three roundings beside it."""
    u = rng.random((N, 3)).astype(np.float32)
    for n in range(0, 3 * N // 4):
        a = n % 3
        x = np.float32(rng.integers(1, order.n_bricks[a])) / np.float32(order.n_bricks[a])
        for _ in range(n // 3 % 4):
            x = np.nextafter(x, np.float32(n // 12 % 2), dtype=np.float32)
        u[n, a] = x
    return u


@pytest.mark.parametrize("key", list(CUTS))
def test_bricks_of_a_large_batch(key):
    """The cuts of large batches on some thousand samples (the calls take a descriptor made for another N), every entry of the
    merged levels against the oracle."""
    print("[case] bricks of a large batch", key, flush=True)
    q = CUTS[key]
    growth = B.dg_growth_factor(16, q["n_max"], 16)
    grid, ref_grid = (f(16, 2, q["log2_T"], 16, growth, q["extent"]) for f in (B.dg_grid_desc_init, oracle.grid_init))
    order = B.dg_order_desc_init(grid, q["made_for"])
    assert list(order.n_bricks) == q["bricks"] and order.n_merged == q["n_merged"] and order.total > 1 << 14
    N, M = 24007, order.n_merged
    rng = np.random.default_rng(36)
    u = _beside_faces(order, N, rng)
    g = (rng.standard_normal((N, 32)) * 1e-3).astype(np.float32)
    ordered = torch.zeros(N, 4, device=DEV)
    pieces = torch.zeros(B.dg_order_pieces_words(order, N), dtype=torch.int32, device=DEV)
    ud, gd = dev(u), dev(_mixed(g, M))
    B.dg_order_samples(order, ud, N, ordered, pieces, torch.zeros(B.dg_order_workspace_bytes(order) // 4, dtype=torch.int32, device=DEV))
    assert np.array_equal(np.sort(host(ordered)[:, 3].copy().view(np.uint32)), np.arange(N))
    dtable = torch.zeros(ref_grid.n_entries, 2, device=DEV)
    ws = torch.zeros(B.dg_hashgrid_encode_bwd_ordered_workspace_bytes(grid, order, N) // 4 + 64, device=DEV)
    B.dg_hashgrid_encode_bwd_ordered(grid, order, ordered, pieces, ud, gd, gd.abs().max().reshape(1).view(torch.int32), N, dtable, ws)
    want = oracle.encode_bwd(ref_grid, u, g.astype(np.float64))
    scale = oracle.encode_bwd(ref_grid, u, np.abs(g).astype(np.float64))
    have = host(dtable).astype(np.float64)
    assert np.all(have[want == 0] == 0)
    quantum = 2.0 ** -37 * float(np.abs(g).max()) * N
    for l in range(M):
        sl = slice(ref_grid.first[l], ref_grid.first[l + 1])
        assert np.all(np.abs(have[sl] - want[sl]) <= 1e-5 * scale[sl] + quantum), l           # bound as in test_ordered_encode
    for l in range(M, 16):
        sl = slice(ref_grid.first[l], ref_grid.first[l + 1])
        assert rel_err(have[sl], want[sl]) <= TOL_F16, l


@pytest.mark.parametrize("N", [1, 21, 64, 127, 1009, 4099])
@pytest.mark.parametrize("n_merged", [2, 4, 6, 8, 10, 12])
def test_every_number_of_merged_levels(n_merged, N):
    """One to six pairs of levels share the wavefronts of a workgroup in different ways, and fewer samples than lanes, one more than a
    piece and everything between divides among them differently.  Three quarters of the samples lie in one brick."""
    print("[case] merged levels", n_merged, N, flush=True)
    q = CUTS["flat"]
    growth = B.dg_growth_factor(16, q["n_max"], 16)
    grid, ref_grid = (f(16, 2, q["log2_T"], 16, growth, q["extent"]) for f in (B.dg_grid_desc_init, oracle.grid_init))
    order = B.dg_order_desc_init(grid, q["made_for"])
    order.n_merged = n_merged
    u = di.make_unit_coords(N, seed=46)
    u[:3 * N // 4] = (np.asarray([0.5, 0.3, 0.4]) + 0.018 * (u[:3 * N // 4] - 0.5)).astype(np.float32)
    g = (np.random.default_rng(47).standard_normal((N, 32)) * 1e-3).astype(np.float32)
    ordered, pieces = torch.zeros(N, 4, device=DEV), torch.zeros(B.dg_order_pieces_words(order, N), dtype=torch.int32, device=DEV)
    ud, gd = dev(u), dev(_mixed(g, n_merged))
    B.dg_order_samples(order, ud, N, ordered, pieces, torch.zeros(B.dg_order_workspace_bytes(order) // 4, dtype=torch.int32, device=DEV))
    dtable = torch.zeros(ref_grid.n_entries, 2, device=DEV)
    ws = torch.zeros(B.dg_hashgrid_encode_bwd_ordered_workspace_bytes(grid, order, N) // 4 + 64, device=DEV)
    B.dg_hashgrid_encode_bwd_ordered(grid, order, ordered, pieces, ud, gd, gd.abs().max().reshape(1).view(torch.int32), N, dtable, ws)
    want, have = oracle.encode_bwd(ref_grid, u, g.astype(np.float64)), host(dtable).astype(np.float64)
    scale = oracle.encode_bwd(ref_grid, u, np.abs(g).astype(np.float64))
    assert np.all(have[want == 0] == 0)
    # four roundings in a contribution, at most eight adds in a lane's run, four over lanes, up to sixteen bricks' into the table
    quantum = 2.0 ** -37 * float(np.abs(g).max()) * N
    for l in range(n_merged):
        sl = slice(ref_grid.first[l], ref_grid.first[l + 1])
        assert np.all(np.abs(have[sl] - want[sl]) <= 32 * 2.0 ** -24 * scale[sl] + quantum), l
    for l in range(n_merged, 16):
        # not the brick sums: records rounded to 2^-20
        sl = slice(ref_grid.first[l], ref_grid.first[l + 1])
        assert np.linalg.norm(have[sl] - want[sl]) <= 4 * 2.0 ** -20 * np.linalg.norm(want[sl]), l


def test_ordered_gradients_of_two_streams_into_one_table():
    """dtable "+=": two streams, each with a workspace of its own, add to one gradient at the same time and nothing of either is lost."""
    print("[case] ordered gradients of two streams", flush=True)
    grid, ref_grid = _grids("large")
    N, passes = 20011, 4
    u = _coords(N, "points")
    order, ordered, pieces = _sorted(grid, u, N)
    g = (np.random.default_rng(48).standard_normal((N, 32)) * 1e-3).astype(np.float32)
    ud, gd = dev(u), dev(_mixed(g, order.n_merged))
    largest = gd.abs().max().reshape(1).view(torch.int32)
    need = B.dg_hashgrid_encode_bwd_ordered_workspace_bytes(grid, order, N) // 4 + 64
    streams, ws = [torch.cuda.Stream() for _ in range(2)], [torch.zeros(need, device=DEV) for _ in range(2)]
    dtable = torch.zeros(ref_grid.n_entries, 2, device=DEV)
    torch.cuda.synchronize()
    for _ in range(passes):
        for s, w in zip(streams, ws):
            with torch.cuda.stream(s):
                B.dg_hashgrid_encode_bwd_ordered(grid, order, ordered, pieces, ud, gd, largest, N, dtable, w)
    torch.cuda.synchronize()
    want, have = 2.0 * passes * oracle.encode_bwd(ref_grid, u, g.astype(np.float64)), host(dtable).astype(np.float64)
    for l in range(16):
        # records rounded to 2^-20, sums rounded to fp32, eight fp32 adds of them
        sl = slice(ref_grid.first[l], ref_grid.first[l + 1])
        assert np.linalg.norm(have[sl] - want[sl]) <= 4 * 2.0 ** -20 * np.linalg.norm(want[sl]), l


@pytest.mark.parametrize("n_merged", [4, 8, 12])
def test_full_pieces_in_one_cell(n_merged):
    """256 bricks whose 4096 samples each lie in one cell of the coarser levels, of either sign: what is added up in fp32 before it
    reaches 64 bits shows here, where no rounding at the end hides it."""
    print("[case] full pieces in one cell", n_merged, flush=True)
    q = CUTS["flat"]
    growth = B.dg_growth_factor(16, q["n_max"], 16)
    grid, ref_grid = (f(16, 2, q["log2_T"], 16, growth, q["extent"]) for f in (B.dg_grid_desc_init, oracle.grid_init))
    order = B.dg_order_desc_init(grid, q["made_for"])
    order.n_merged = n_merged
    rng = np.random.default_rng(49)
    N, bricks = 256 * 4096, rng.choice(order.total, 256, replace=False)
    nx, ny, nz = order.n_bricks
    middle = (np.stack([bricks % nx, bricks // nx % ny, bricks // (nx * ny)], 1) + 0.5) / np.asarray([nx, ny, nz])
    u = (np.repeat(middle, 4096, 0) + 1e-3 * (rng.random((N, 3)) - 0.5)).astype(np.float32)
    g = np.zeros((N, 32), np.float32)
    g[:, :2 * n_merged] = rng.standard_normal((N, 2 * n_merged)) * 1e-3
    ordered, pieces = torch.zeros(N, 4, device=DEV), torch.zeros(B.dg_order_pieces_words(order, N), dtype=torch.int32, device=DEV)
    ud, gd = dev(u), dev(_mixed(g, n_merged))
    B.dg_order_samples(order, ud, N, ordered, pieces, torch.zeros(B.dg_order_workspace_bytes(order) // 4, dtype=torch.int32, device=DEV))
    assert int(pieces[0]) == 256
    dtable = torch.zeros(ref_grid.n_entries, 2, device=DEV)
    ws = torch.zeros(B.dg_hashgrid_encode_bwd_ordered_workspace_bytes(grid, order, N) // 4 + 64, device=DEV)
    B.dg_hashgrid_encode_bwd_ordered(grid, order, ordered, pieces, ud, gd, gd.abs().max().reshape(1).view(torch.int32), N, dtable, ws)
    want, have = oracle.encode_bwd(ref_grid, u, g.astype(np.float64)), host(dtable).astype(np.float64)
    for l in range(n_merged):
        sl = slice(ref_grid.first[l], ref_grid.first[l + 1])
        # terms of either sign: roundings add up in quadrature, and so do the terms to `want`.  Per sample four in the contribution, 7.5 on
        # average in the sums over samples and lanes, and the last to fp32 and its adds: 13 of 0.42 x 2^-24 each (a rounding is uniform
        # over an ulp, which is 2^-24 to 2^-23 of the value), 9.0e-8; 512 bricks and features to average over: 11 % for three deviations
        assert np.linalg.norm(have[sl] - want[sl]) <= 1.0e-7 * np.linalg.norm(want[sl]), l


def test_many_bricks_to_an_entry():
    """29 791 bricks on tables of 2^14 entries: some seventy bricks and more add to an entry.  Their sums are added in fp64, so what is
    left are the roundings of a contribution (two products for its weight, one with the gradient, one of 1 - fraction) and that of the
    entry: five independent ones of at most 2^-24, sqrt(5 / 3) 2^-24 = 7.7e-8 in 2-norm (with fp32 adds 1.3e-7 to 1.8e-7)."""
    print("[case] many bricks to an entry", flush=True)
    growth = B.dg_growth_factor(16, 1024, 16)
    grid, ref_grid = (f(16, 2, 14, 16, growth, [1.0, 1.0, 1.0]) for f in (B.dg_grid_desc_init, oracle.grid_init))
    order = B.dg_order_desc_init(grid, 1 << 26)
    N, M = 200003, order.n_merged
    assert order.total == 29791 and M >= 8
    u = di.make_unit_coords(N, seed=38)
    g = (np.random.default_rng(39).standard_normal((N, 32)) * 1e-3).astype(np.float32)
    ordered, pieces = torch.zeros(N, 4, device=DEV), torch.zeros(B.dg_order_pieces_words(order, N), dtype=torch.int32, device=DEV)
    ud, gd = dev(u), dev(_mixed(g, M))
    B.dg_order_samples(order, ud, N, ordered, pieces, torch.zeros(B.dg_order_workspace_bytes(order) // 4, dtype=torch.int32, device=DEV))
    dtable = torch.zeros(ref_grid.n_entries, 2, device=DEV)
    ws = torch.zeros(B.dg_hashgrid_encode_bwd_ordered_workspace_bytes(grid, order, N) // 4 + 64, device=DEV)
    B.dg_hashgrid_encode_bwd_ordered(grid, order, ordered, pieces, ud, gd, gd.abs().max().reshape(1).view(torch.int32), N, dtable, ws)
    want, have = oracle.encode_bwd(ref_grid, u, g.astype(np.float64)), host(dtable).astype(np.float64)
    off = [float(np.linalg.norm(have[a:b] - want[a:b]) / np.linalg.norm(want[a:b])) for a, b in zip(ref_grid.first[:M], ref_grid.first[1:M + 1])]
    print("[case] 2-norms", ["%.1e" % x for x in off], flush=True)
    assert max(off) <= (5.0 / 3.0) ** 0.5 * 2.0 ** -24


@pytest.mark.parametrize("flavour", FLAVOURS)
@pytest.mark.parametrize("log2_T", [11, 14, 17, 20, 22, 23, 24])
def test_unmerged_levels_of_every_table_size(log2_T, flavour):
    """Levels of up to 2048 bins, the last step partly filled; with all samples in a few cells most records find their ring full.  Pairs whose
    entries lie in different bins are among them.  T = 2^11 and 2^14 have so few bins that all are summed directly; from 2^17 on queues are
    filled from rings of 128 lines to one (test_queues_of_few_bins: longer ones)."""
    print("[case] unmerged levels", log2_T, flavour, flush=True)
    growth = B.dg_growth_factor(16, 1024, 16)
    grid, ref_grid = (f(16, 2, log2_T, 16, growth, [1.0, 0.9, 0.5]) for f in (B.dg_grid_desc_init, oracle.grid_init))
    N = 150001
    u = _coords(N, flavour)
    order, ordered, pieces = _sorted(grid, u, N)
    M = order.n_merged
    assert M < 12 and max(ref_grid.first[l + 1] - ref_grid.first[l] for l in range(M, 16)) == 1 << log2_T
    g = (np.random.default_rng(50).standard_normal((N, 32)) * 1e-3).astype(np.float32)
    g[5::11] = 0.0
    gd = dev(_mixed(g, M))
    dtable = torch.zeros(ref_grid.n_entries, 2, device=DEV)
    ws = torch.full((B.dg_hashgrid_encode_bwd_ordered_workspace_bytes(grid, order, N) // 4 + 64,), float("nan"), device=DEV)
    B.dg_hashgrid_encode_bwd_ordered(grid, order, ordered, pieces, dev(u), gd, gd.abs().max().reshape(1).view(torch.int32), N, dtable, ws)
    want, have = oracle.encode_bwd(ref_grid, u, g.astype(np.float64)), host(dtable).astype(np.float64)
    scale = oracle.encode_bwd(ref_grid, u, np.abs(g).astype(np.float64))
    for l in range(M, 16):
        # every contribution is rounded to 2^-19 of itself at most and is four fp32 roundings deep, an x fraction to 2^-24, the sum to fp32.  Samples
        # all over the box also average: a rounding is uniform, 2^-19 / sqrt(3) = 1.1e-6 in 2-norm, and few terms meet in an entry
        sl = slice(ref_grid.first[l], ref_grid.first[l + 1])
        off = np.linalg.norm(have[sl] - want[sl])
        assert np.all(have[sl][want[sl] == 0] == 0), l
        assert off <= (2.0 ** -19 + 8 * 2.0 ** -24) * np.linalg.norm(scale[sl]), l
        if flavour == "points":
            assert off <= 1.2e-6 * np.linalg.norm(want[sl]), l


@pytest.mark.parametrize("log2_T", [17, 22, 24])
def test_fractions_finer_than_a_record(log2_T):
    """Samples next to a face of the first cell along x, where the fp32 fraction has more bits than the record's 2^-23 of a cell: every entry,
    also those that only such samples touch, is as good as its 27-bit values.  Hashed levels (T = 2^17), dense ones among them (2^24)."""
    print("[case] first cell along x", log2_T, flush=True)
    growth = B.dg_growth_factor(16, 1024, 16)
    grid, ref_grid = (f(16, 2, log2_T, 16, growth, [1.0, 0.9, 0.5]) for f in (B.dg_grid_desc_init, oracle.grid_init))
    N = 150001
    rng = np.random.default_rng(53)
    u = _coords(N, "points")
    order = B.dg_order_desc_init(grid, N)
    M = order.n_merged
    level = rng.integers(M, 16, N)
    scale = np.asarray([grid.scale[l][0] for l in range(16)])[level]
    near_0, near_1 = 2.0 ** rng.uniform(-26, 0, N), 1.0 - rng.integers(1, 1 << 10, N) * 2.0 ** -24
    u[:, 0] = np.where(rng.random(N) < 0.7, near_0, near_1) / scale
    order, ordered, pieces = _sorted(grid, u, N)
    assert order.n_merged == M
    g = ((0.5 + rng.random((N, 32))) * rng.choice([-1e-3, 1e-3], (N, 32))).astype(np.float32)
    gd = dev(_mixed(g, M))
    dtable = torch.zeros(ref_grid.n_entries, 2, device=DEV)
    ws = torch.full((B.dg_hashgrid_encode_bwd_ordered_workspace_bytes(grid, order, N) // 4 + 64,), float("nan"), device=DEV)
    B.dg_hashgrid_encode_bwd_ordered(grid, order, ordered, pieces, dev(u), gd, gd.abs().max().reshape(1).view(torch.int32), N, dtable, ws)
    want, have = oracle.encode_bwd(ref_grid, u, g.astype(np.float64)), host(dtable).astype(np.float64)
    magnitude = oracle.encode_bwd(ref_grid, u, np.abs(g).astype(np.float64))
    idx = torch.zeros(N, 16, 8, dtype=torch.int32, device=DEV)
    B.dg_hashgrid_corner_indices(grid, dev(u), N, idx)
    records = host(torch.bincount(idx.reshape(-1), minlength=ref_grid.n_entries)).astype(np.float64)[:, None]
    # a value keeps 18 mantissa bits (half a unit: 2^-19), its x fraction is off by 2^-21 of the share at most, it is five fp32 roundings deep, the sum's and those of the adds past the queues
    # (partial sums of terms of either sign) are below three more; half a quantum of 2^-31 of the largest magnitude per add, of which a corner
    # whose pair goes apart takes two
    bound = (2.0 ** -19 + 2.0 ** -21 + 8 * 2.0 ** -24) * magnitude + 2.0 ** -31 * float(np.abs(g).max()) * records
    for l in range(M, 16):
        sl = slice(ref_grid.first[l], ref_grid.first[l + 1])
        worst = np.abs(have[sl] - want[sl]) / np.maximum(bound[sl], 1e-300)
        print("[case] level", l, "dense" if grid.dense[l] else "hashed", "worst %.2f of the bound" % worst[magnitude[sl] > 0].max(), flush=True)
    for l in range(M, 16):
        sl = slice(ref_grid.first[l], ref_grid.first[l + 1])
        assert np.all(np.abs(have[sl] - want[sl]) <= bound[sl]), l


@pytest.mark.parametrize("flavour", FLAVOURS)
@pytest.mark.parametrize("log2_T", [14, 20, 22, 23, 24])
def test_ray_order_queues_of_every_table_size(log2_T, flavour):
    """The same for samples in the order of their rays: records of merged runs, four in a line, and rings of half as many lines for up to 512
    bins.  T = 2^14 is summed directly."""
    print("[case] ray order", log2_T, flavour, flush=True)
    growth = B.dg_growth_factor(16, 1024, 16)
    grid, ref_grid = (f(16, 2, log2_T, 16, growth, [1.0, 0.9, 0.5]) for f in (B.dg_grid_desc_init, oracle.grid_init))
    N = 150001
    u = _coords(N, flavour)
    g = (np.random.default_rng(51).standard_normal((N, 32)) * 1e-3).astype(np.float32)
    g[5::11] = 0.0
    gd = dev(np.ascontiguousarray(g.reshape(N, 16, 2).transpose(1, 0, 2)))
    dtable = torch.zeros(ref_grid.n_entries, 2, device=DEV)
    ws = torch.full((B.dg_hashgrid_encode_bwd_workspace_bytes(grid, N) // 4 + 64,), float("nan"), device=DEV)
    B.dg_hashgrid_encode_bwd(grid, dev(u), gd, N, dtable, ws)
    want, have = oracle.encode_bwd(ref_grid, u, g.astype(np.float64)), host(dtable).astype(np.float64)
    scale = oracle.encode_bwd(ref_grid, u, np.abs(g).astype(np.float64))
    for l in range(16):
        # a contribution is four fp32 roundings deep, a run of up to 64 adds six more, a record rounds to 2^-19 at most, and the bin's flush to fp32
        sl = slice(ref_grid.first[l], ref_grid.first[l + 1])
        assert np.all(have[sl][want[sl] == 0] == 0), l
        assert np.linalg.norm(have[sl] - want[sl]) <= (2.0 ** -19 + 14 * 2.0 ** -24) * np.linalg.norm(scale[sl]), l


@pytest.mark.parametrize("flavour", FLAVOURS)
@pytest.mark.parametrize("spatial", [False, True])
@pytest.mark.parametrize("log2_T,n_max,N,merged,fewest,most", [(18, 64, 150001, 2, 1, 16), (15, 1024, 400001, None, 4, 4)])
def test_queues_of_few_bins(log2_T, n_max, N, merged, fewest, most, spatial, flavour):
    """Levels of one to sixteen bins and of four that go through queues all the same: rings of 2048 (in ray order 1024) lines to 128 (64), written out by as
    many groups of lanes to a bin as there are."""
    print("[case] few bins", log2_T, n_max, spatial, flavour, flush=True)
    extent, growth = [1.0, 0.9, 0.5], B.dg_growth_factor(16, n_max, 16)
    grid, ref_grid = (f(16, 2, log2_T, 16, growth, extent) for f in (B.dg_grid_desc_init, oracle.grid_init))
    u = _coords(N, flavour)
    order, ordered, pieces = _sorted(grid, u, N)
    if merged is not None:
        order.n_merged = merged
    M = order.n_merged if spatial else 0
    first = max(M, sum(e <= 8192 for e in ref_grid.first[1:17]))            # the levels below have a way of their own
    have_bins = [-((ref_grid.first[l] - ref_grid.first[l + 1]) // 8192) for l in range(first, 16)]
    assert min(have_bins) <= fewest and max(have_bins) == most
    g = (np.random.default_rng(54).standard_normal((N, 32)) * 1e-3).astype(np.float32)
    ud, need = dev(u), (B.dg_hashgrid_encode_bwd_ordered_workspace_bytes(grid, order, N) if spatial else B.dg_hashgrid_encode_bwd_workspace_bytes(grid, N))

    def gradient(planes_of):
        gd, dtable, ws = dev(_mixed(planes_of, M)), torch.zeros(ref_grid.n_entries, 2, device=DEV), torch.full((need // 4 + 64,), float("nan"), device=DEV)
        if spatial:
            B.dg_hashgrid_encode_bwd_ordered(grid, order, ordered, pieces, ud, gd, dev(np.abs(g).max().reshape(1)).view(torch.int32), N, dtable, ws)
        else:
            B.dg_hashgrid_encode_bwd(grid, ud, gd, N, dtable, ws)
        return host(dtable)

    # an infinite gradient at the first of these levels marks every bin of a queue, and its own entries alone where bins are summed directly
    marked = g.copy()
    marked[0, 2 * first] = np.inf
    assert not np.isfinite(gradient(marked)[ref_grid.first[15]:]).all()
    want, have = oracle.encode_bwd(ref_grid, u, g.astype(np.float64)), gradient(g).astype(np.float64)
    scale = oracle.encode_bwd(ref_grid, u, np.abs(g).astype(np.float64))
    for l in range(first, 16):
        # as in test_ray_order_queues_of_every_table_size; half a quantum of 2^-31 of the largest sum of a run, which some thousands of records share
        sl = slice(ref_grid.first[l], ref_grid.first[l + 1])
        assert np.all(have[sl][want[sl] == 0] == 0), l
        assert np.linalg.norm(have[sl] - want[sl]) <= (2.0 ** -19 + 14 * 2.0 ** -24) * np.linalg.norm(scale[sl]), l


@pytest.mark.parametrize("spatial", [False, True])
@pytest.mark.parametrize("log2_T,n_max,room", [(20, 2048, 18933760), (22, 2048, 64 << 20), (22, 8192, 64 << 20)])
def test_gradient_through_a_small_workspace(log2_T, n_max, room, spatial):
    """Levels of 128 and of 512 bins in less room than all workgroups' slices of them would take up with their last lines alone: batches, the last
    one partly filled, against the sums of one batch."""
    print("[case] small workspace", log2_T, n_max, room, spatial, flush=True)
    growth = B.dg_growth_factor(16, n_max, 16)
    grid, ref_grid = (f(16, 2, log2_T, 16, growth, [2.0, 2.0, 0.25]) for f in (B.dg_grid_desc_init, oracle.grid_init))
    N = 150001
    u = _coords(N, "points")
    order, ordered, pieces = _sorted(grid, u, N)
    M = order.n_merged if spatial else 0
    g = (np.random.default_rng(52).standard_normal((N, 32)) * 1e-3).astype(np.float32)
    gd = dev(_mixed(g, M))
    dtable, ws = torch.zeros(ref_grid.n_entries, 2, device=DEV), torch.full((room // 4,), float("nan"), device=DEV)
    if spatial:
        assert room < B.dg_hashgrid_encode_bwd_ordered_workspace_bytes(grid, order, N)
        B.dg_hashgrid_encode_bwd_ordered(grid, order, ordered, pieces, dev(u), gd, gd.abs().max().reshape(1).view(torch.int32), N, dtable, ws)
    else:
        assert room < B.dg_hashgrid_encode_bwd_workspace_bytes(grid, N)
        B.dg_hashgrid_encode_bwd(grid, dev(u), gd, N, dtable, ws)
    want, have = oracle.encode_bwd(ref_grid, u, g.astype(np.float64)), host(dtable).astype(np.float64)
    scale = oracle.encode_bwd(ref_grid, u, np.abs(g).astype(np.float64))
    for l in range(16):
        # as for one batch (test_ray_order_queues_of_every_table_size), and each of up to sixteen batches adds to an entry in fp32
        sl = slice(ref_grid.first[l], ref_grid.first[l + 1])
        assert np.all(have[sl][want[sl] == 0] == 0), l
        assert np.linalg.norm(have[sl] - want[sl]) <= (2.0 ** -19 + 30 * 2.0 ** -24) * np.linalg.norm(scale[sl]), l


@pytest.mark.parametrize("N,log2_T,n_max", [((1 << 22) + 77, 19, 2048), ((1 << 21) + 5, 22, 8192)])
def test_ordered_gradient_at_full_size(N, log2_T, n_max):
    """A batch of production size, level by level and entry by entry against the pass in ray order on the same gradient."""
    print("[case] ordered gradient at full size", N, log2_T, flush=True)
    grid = B.dg_grid_desc_init(16, 2, log2_T, 16, B.dg_growth_factor(16, n_max, 16), [2.0, 2.0, 0.25])
    gen = torch.Generator(device=DEV)
    gen.manual_seed(37)
    u = torch.rand(N, 3, device=DEV, generator=gen)
    planes = torch.randn(16, N, 2, device=DEV, generator=gen) * 1e-3
    order = B.dg_order_desc_init(grid, N)
    M = order.n_merged
    ordered, pieces = torch.zeros(N, 4, device=DEV), torch.zeros(B.dg_order_pieces_words(order, N), dtype=torch.int32, device=DEV)
    B.dg_order_samples(order, u, N, ordered, pieces, torch.zeros(B.dg_order_workspace_bytes(order) // 4, dtype=torch.int32, device=DEV))
    mixed = torch.cat([planes[:M].transpose(0, 1).reshape(-1), planes[M:].reshape(-1)])
    ws = torch.zeros(B.dg_hashgrid_encode_bwd_workspace_bytes(grid, N) // 4 + 64, device=DEV)
    got, want, scale = (torch.zeros(grid.n_entries, 2, device=DEV) for _ in range(3))
    B.dg_hashgrid_encode_bwd_ordered(grid, order, ordered, pieces, u, mixed, mixed.abs().max().reshape(1).view(torch.int32), N, got, ws)
    B.dg_hashgrid_encode_bwd(grid, u, planes, N, want, ws)
    B.dg_hashgrid_encode_bwd(grid, u, planes.abs(), N, scale, ws)
    for l in range(16):
        sl = slice(grid.offset[l], grid.offset[l + 1])
        # in ray order a value is rounded to 2^-20 (both paths at the unmerged levels), to a quantum of 2^-31 of the largest per record
        # and reaches the table by a handful of fp32 adds; the ordered side is below 1e-5 as in test_ordered_encode
        assert bool(((got[sl] - want[sl]).abs() <= 1.5e-5 * scale[sl] + 2.0 ** -31 * 8e-3 * 64).all()), l
        assert float((got[sl] - want[sl]).norm() / want[sl].norm()) <= 4 * 2.0 ** -20, l


@pytest.mark.parametrize("bad", ["overflow", "nan", None])
def test_largest_gradient_of_the_networks(bad):
    """The word that the networks report for the brick sums: the largest magnitude of what they write, infinity where a delta
    overflows fp16 or is NaN; the table gradient that follows is then marked at every merged level."""
    print("[case] largest gradient", bad, flush=True)
    grid, ref_grid = _grids("cached")
    N = 3001
    mlp = B.dg_mlp_desc(32, 64, 16, 16, 64, 2, 1)
    rng = np.random.default_rng(44)
    u = _coords(N, "points")
    order, ordered, pieces = _sorted(grid, u, N)
    M = order.n_merged
    rows = torch.zeros(N, 32, dtype=torch.float16, device=DEV)
    B.dg_hashgrid_encode_fwd_ordered(grid, dev(di.make_table(ref_grid.n_entries, 2, 1.0, seed=45)), ordered, N, rows)
    dsigma, drgb = dev((rng.standard_normal(N) * 1e-4).astype(np.float32)), dev((rng.standard_normal((N, 3)) * 1e-4).astype(np.float32))
    if bad == "nan":
        dsigma[1234] = float("nan")
    weights, dir_enc = dev((rng.standard_normal(9408) * 0.2).astype(np.float16)), torch.zeros(-(-N // 32), 16, dtype=torch.float16, device=DEV)
    dfeat, dW = torch.zeros(N * 32, device=DEV), torch.zeros(9408, device=DEV)
    largest = pieces[1:2]
    assert int(largest) == 0
    B.dg_mlp_bwd_rows(mlp, weights, rows, dir_enc, None, 32, N, dsigma, drgb, 2.0 ** (60 if bad == "overflow" else 12), M, dfeat, largest, dW,
                      torch.zeros(B.dg_mlp_bwd_app_workspace_bytes(mlp, N, 32) // 4 + 64, device=DEV))
    reported = float(largest.view(torch.float32))
    if bad is None:
        assert reported == float(dfeat.abs().max()) > 0
    else:
        assert reported == float("inf")
    dtable = torch.zeros(ref_grid.n_entries, 2, device=DEV)
    ws = torch.zeros(B.dg_hashgrid_encode_bwd_ordered_workspace_bytes(grid, order, N) // 4 + 64, device=DEV)
    B.dg_hashgrid_encode_bwd_ordered(grid, order, ordered, pieces, dev(u), dfeat, largest, N, dtable, ws)
    for l in range(M):
        assert bool(torch.isfinite(dtable[ref_grid.first[l]:ref_grid.first[l + 1]]).all()) == (bad is None), l


def test_non_finite_gradient_is_marked():
    """An infinite or NaN gradient (an fp16 delta that overflowed) leaves NaN in the table gradient's merged levels."""
    grid, ref_grid = _grids("cached")
    N = 3000
    u = _coords(N, "points")
    order, ordered, pieces = _sorted(grid, u, N)
    ws = torch.zeros(B.dg_hashgrid_encode_bwd_ordered_workspace_bytes(grid, order, N) // 4 + 64, device=DEV)
    for bad in (float("inf"), float("nan")):
        g = torch.zeros(N * 32, device=DEV)
        g[5] = bad
        dtable = torch.zeros(ref_grid.n_entries, 2, device=DEV)
        largest = torch.tensor([float("inf")], device=DEV).view(torch.int32)         # what dg_mlp_bwd_rows reports for either
        B.dg_hashgrid_encode_bwd_ordered(grid, order, ordered, pieces, dev(u), g, largest, N, dtable, ws)
        assert not bool(torch.isfinite(dtable).all())


def test_order_arguments():
    grid, _ = _grids("cached")
    order = B.dg_order_desc_init(grid, 5000)
    u, ordered = torch.rand(5000, 3, device=DEV), torch.zeros(5000, 4, device=DEV)
    pieces = torch.zeros(B.dg_order_pieces_words(order, 5000), dtype=torch.int32, device=DEV)
    with pytest.raises(B.DistGridError):                                                 # workspace too small
        B.dg_order_samples(order, u, 5000, ordered, pieces, torch.zeros(8, dtype=torch.int32, device=DEV))
    shallow = B.dg_grid_desc_init(4, 2, 12, 16, 1.5, [1.0, 1.0, 1.0])
    with pytest.raises(B.DistGridError):
        B.dg_order_desc_init(shallow, 5000)


@pytest.mark.parametrize("name,R,overrides", [("c2_ngp", 1500, {}), ("c3_2x2", 1200, dict(log2_T=16)), ("c8_app", 700, {})])
def test_step_in_spatial_order(name, R, overrides, monkeypatch):
    """The training step with the order forced at a small size, through every comparison of the plain step."""
    from test_gpu_step import _compare_step
    print("[case] step in spatial order", name, R, flush=True)
    monkeypatch.setattr(TrainStep, "_order_min", lambda self, m: 1)
    cfg = di.config(name)
    cfg["grid"] = dict(cfg["grid"], **overrides)
    step, _ = _compare_step(cfg, R, seed=2, lambda1=1e-3, loss_scale=2.0 ** 14, use_jitter_array=False, table_gain=3000.0)
    assert all(order is not None for _, _, order in step.layout.values())


def test_cascade_in_spatial_order(monkeypatch):
    """The two-level cascade with the order forced: eight sub-models, regions with holes, rays that meet a sub-model twice."""
    from test_gpu_step import _compare_step
    print("[case] cascade in spatial order", flush=True)
    monkeypatch.setattr(TrainStep, "_order_min", lambda self, m: 1)
    cfg = di.config("c6_cascade")
    cfg["grid"], cfg["grid_coarse"] = dict(cfg["grid"], log2_T=16), dict(cfg["grid_coarse"], log2_T=14)
    step, _ = _compare_step(cfg, 700, seed=7, lambda1=1e-3, loss_scale=2.0 ** 14, use_jitter_array=False, table_gain=3000.0)
    assert len(step.layout) == 8 and all(order is not None for _, _, order in step.layout.values())


@pytest.mark.parametrize("name,R,room", [("c7_occ", 1100, 60000), ("c3_2x2", 800, 200000)])
def test_occupancy_step_in_spatial_order(name, R, room, monkeypatch):
    """Occupancy-guided samples with the order forced: segments of different lengths, one box and four."""
    from test_gpu_step_occupancy import _compare
    print("[case] occupancy step in spatial order", name, flush=True)
    monkeypatch.setattr(TrainStep, "_order_min", lambda self, m: 1)
    cfg = di.config(name)
    cfg["occ"] = dict(res=48, max_steps=512)
    cfg["grid"] = dict(cfg["grid"], log2_T=16)
    step, ref = _compare(cfg, R, seed=3, lambda1=1e-3, loss_scale=2.0 ** 14, table_gain=3000.0, max_samples=room)
    assert len(step.layout) == len(ref["per"]) and all(order is not None for _, _, order in step.layout.values())


def test_step_without_mergeable_levels(monkeypatch):
    """A grid whose coarsest levels do not fit LDS brick by brick: served by the plain kernels, whatever the batch size."""
    from test_gpu_step import _compare_step
    print("[case] step without mergeable levels", flush=True)
    monkeypatch.setattr(TrainStep, "_order_min", lambda self, m: 1)
    cfg = di.config("c2_ngp")
    cfg["grid"] = dict(cfg["grid"], n_min=600, n_max=2048, growth=None, log2_T=15)
    step, _ = _compare_step(cfg, 300, seed=2, lambda1=1e-3, loss_scale=2.0 ** 14, use_jitter_array=False, table_gain=3000.0)
    assert all(order is None for _, _, order in step.layout.values())


def test_render_in_spatial_order(monkeypatch):
    from gpu_util import gpu_models, make_step
    import oracle.step as ostep
    cfg = di.config("c2_ngp", table_range=0.3)
    R = 801
    o, d = di.make_rays(cfg, seed=5, R=R)
    hm = ostep.make_models(cfg, seed=5)
    plain = make_step(cfg, gpu_models(cfg, hm), R, seed=5)
    monkeypatch.setattr(TrainStep, "_order_min", lambda self, m: 1)
    sorted_ = make_step(cfg, gpu_models(cfg, hm), R, seed=5)
    for fused in (None, False):
        want = [x.clone() for x in plain.render(dev(o), dev(d), fused=fused)]
        got = sorted_.render(dev(o), dev(d), fused=fused)
        assert sorted_.layout[0][2] is not None
        for a, b in zip(got, want):
            assert rel_err(host(a), host(b)) <= TOL_F16


@pytest.mark.parametrize("N", [1, 31, 33, 5003])
def test_density_of_candidates(N):
    """Density net and maximum in one kernel, planes and sorted rows, against the separate entry points: the same bits."""
    print("[case] density of candidates", N, flush=True)
    grid, ref_grid = _grids("cached")
    mlp = B.dg_mlp_desc(32, 64, 16, 16, 64, 2, 1)
    rng = np.random.default_rng(41)
    table = dev(di.make_table(ref_grid.n_entries, 2, 1.0, seed=42))
    weights = dev((rng.standard_normal(9408) * 0.2).astype(np.float16))
    n_cells = 700
    u, cell = dev(_coords(N, "points")), torch.from_numpy(rng.integers(0, n_cells + 50, N).astype(np.int32)).to(DEV)     # some past the grid: left out
    planes, sigma, rgb = torch.zeros(N, 32, dtype=torch.float16, device=DEV), torch.zeros(N, device=DEV), torch.zeros(N, 3, device=DEV)
    B.dg_hashgrid_encode_fwd(grid, table, u, N, planes)
    B.dg_mlp_fwd(mlp, weights, planes, torch.zeros(1, 16, dtype=torch.float16, device=DEV), N, N, sigma, rgb)
    start = torch.rand(n_cells, device=DEV)
    want = start.clone()
    B.dg_occ_update(want, cell, sigma, N)
    got = start.clone()
    B.dg_occ_evaluate(mlp, weights, planes, False, cell, 1, N, got)
    assert torch.equal(got, want)
    order = B.dg_order_desc_init(grid, N)
    ordered, rows = torch.zeros(N, 4, device=DEV), torch.zeros(N, 32, dtype=torch.float16, device=DEV)
    pieces = torch.zeros(B.dg_order_pieces_words(order, N), dtype=torch.int32, device=DEV)
    ws = torch.zeros(B.dg_order_workspace_bytes(order) // 4, dtype=torch.int32, device=DEV)
    B.dg_order_samples(order, u, N, ordered, pieces, ws, ids=cell)
    assert torch.equal(ordered[:, 3].contiguous().view(torch.int32).sort().values, cell.sort().values)
    B.dg_hashgrid_encode_fwd_ordered(grid, table, ordered, N, rows, by_position=True)
    got = start.clone()
    B.dg_occ_evaluate(mlp, weights, rows, True, ordered.view(-1)[3:4 * N].view(torch.int32), 4, N, got)
    # the two encodes add a cell's corners up in another order, so features differ by fp32 rounding before theirs to fp16
    assert rel_err(host(got), host(want)) <= TOL_F16
    small = B.dg_mlp_desc(8, 32, 16, 4, 32, 1, 1)
    with pytest.raises(B.DistGridError):
        B.dg_occ_evaluate(small, weights, planes, False, cell, 1, N, got)


@pytest.mark.parametrize("n_app", [0, 48])
@pytest.mark.parametrize("key,N", [(key, N) for key in GRIDS for N in (1, 31, 63, 1025, 20011)])
def test_split_features(key, N, n_app):
    """Features as rows of twelve levels and planes of four: the ordered gather's features level by level, and from them the networks'
    results of the features in rows, forward, backward and of candidates."""
    print("[case] split features", key, N, n_app, flush=True)
    grid, ref_grid = _grids(key)
    rng = np.random.default_rng(46)
    u = _coords(N, "faces")
    order, ordered, _ = _sorted(grid, u, N)
    table, ud = dev(di.make_table(ref_grid.n_entries, 2, 1.0, seed=47)), dev(u)
    rows, split = (torch.full((N, 32), float("nan"), dtype=torch.float16, device=DEV) for _ in range(2))
    for by_position in (True, False):                   # the last one's are the samples' own order
        B.dg_hashgrid_encode_fwd_ordered(grid, table, ordered, N, rows, by_position=by_position)
        B.dg_hashgrid_encode_fwd_split(grid, table, ordered, ud, N, split, by_position=by_position)
        flat, n_rows = split.view(-1), 2 * B.SPLIT_LEVELS * N
        assert torch.equal(flat[:n_rows].view(N, -1), rows[:, :2 * B.SPLIT_LEVELS])
        assert torch.equal(flat[n_rows:].view(-1, N, 2).transpose(0, 1).reshape(N, -1), rows[:, 2 * B.SPLIT_LEVELS:])
        if by_position:
            mlp = B.dg_mlp_desc(32, 64, 16, 16, 64, 2, 1)
            weights = dev((rng.standard_normal(9408) * 0.2).astype(np.float16))
            cell, got, want = torch.arange(N, dtype=torch.int32, device=DEV), torch.zeros(N, device=DEV), torch.zeros(N, device=DEV)
            B.dg_occ_evaluate_split(mlp, weights, split, cell, 1, N, got)
            B.dg_occ_evaluate(mlp, weights, rows, True, cell, 1, N, want)
            assert torch.equal(got, want)

    mlp, S = B.dg_mlp_desc(32, 64, 16, 16, 64, 2, 1, n_app=n_app), 37
    weights = dev((rng.standard_normal(B.dg_mlp_weight_count(mlp)) * 0.2).astype(np.float16))
    n_dir = -(-N // S)
    dir_enc = dev(rng.standard_normal((n_dir, 16)).astype(np.float16))
    app = dev(rng.standard_normal((n_dir, n_app)).astype(np.float16)) if n_app else None
    dsigma, drgb = dev((rng.standard_normal(N) * 1e-4).astype(np.float32)), dev((rng.standard_normal((N, 3)) * 1e-4).astype(np.float32))
    ws = torch.zeros(B.dg_mlp_bwd_app_workspace_bytes(mlp, N, S) // 4 + 64, device=DEV)
    results = []
    for fwd, bwd, feat in ((B.dg_mlp_fwd_rows, B.dg_mlp_bwd_rows, rows), (B.dg_mlp_fwd_split, B.dg_mlp_bwd_split, split)):
        sigma, rgb, dfeat = torch.zeros(N, device=DEV), torch.zeros(N, 3, device=DEV), torch.zeros(N * 32, device=DEV)
        dW, largest = torch.zeros(B.dg_mlp_weight_count(mlp), device=DEV), torch.zeros(1, dtype=torch.int32, device=DEV)
        fwd(mlp, weights, feat, dir_enc, app, S, N, sigma, rgb)
        bwd(mlp, weights, feat, dir_enc, app, S, N, dsigma, drgb, 4096.0, order.n_merged, dfeat, largest, dW, ws)
        results.append((sigma, rgb, dfeat, largest, dW[:9408], dW[9408:]))
    for a, b in list(zip(*results))[:5]:                # one kernel on the same numbers read from other places
        assert torch.equal(a, b)
    # the appearance columns' sums go out by fp32 atomics, one per column and tile, in any order: each add rounds by 2^-24 of a partial sum
    # no larger than sqrt(tiles) typical terms in random signs, tiles of them
    assert not n_app or rel_err(host(results[1][5]), host(results[0][5])) <= 2.0 ** -24 * max(-(-N // 32), 1)


@pytest.mark.parametrize("by_position", [False, True])
@pytest.mark.parametrize("n_merged", [6, 8, 10, 12])
@pytest.mark.parametrize("key,N", [(key, N) for key in ("flat", "cube", "upright") for N in (1, 513, 4097, 24007)])
def test_features_brick_by_brick(key, N, n_merged, by_position):
    """Levels gathered from a brick's vertices in LDS: samples on the bricks' faces and up to three roundings beside them, in corners of the box
    and outside it, and one brick that holds several pieces."""
    print("[case] features brick by brick", key, N, n_merged, by_position, flush=True)
    q = CUTS[key]
    growth = B.dg_growth_factor(16, q["n_max"], 16)
    grid, ref_grid = (f(16, 2, q["log2_T"], 16, growth, q["extent"]) for f in (B.dg_grid_desc_init, oracle.grid_init))
    order = B.dg_order_desc_init(grid, q["made_for"])
    order.n_merged = min(n_merged, order.n_merged)
    u = _beside_faces(order, N, np.random.default_rng(51))
    u[:5] = np.asarray([[0, 0, 0], [1, 1, 1], [-0.3, 0.5, 2.0], [1, 0, 0.5], [0.99999994, 0.5, 0.0]], np.float32)[:N]
    u[N // 2:] = (np.asarray([0.5, 0.3, 0.4]) + 4e-3 * (u[N // 2:] - 0.5)).astype(np.float32)          # half of them in one brick or two
    ordered, pieces = torch.zeros(N, 4, device=DEV), torch.zeros(B.dg_order_pieces_words(order, N), dtype=torch.int32, device=DEV)
    ud, table = dev(u), di.make_table(ref_grid.n_entries, 2, 1.0, seed=52)
    B.dg_order_samples(order, ud, N, ordered, pieces, torch.zeros(B.dg_order_workspace_bytes(order) // 4, dtype=torch.int32, device=DEV))
    feat = torch.full((N, 32), float("nan"), dtype=torch.float16, device=DEV)
    B.dg_hashgrid_encode_fwd_bricks(grid, order, dev(table), ordered, pieces, ud, N, feat, by_position=by_position)
    flat, n_rows = host(feat).reshape(-1), 2 * B.SPLIT_LEVELS * N
    got = np.concatenate([flat[:n_rows].reshape(N, -1), flat[n_rows:].reshape(-1, N, 2).transpose(1, 0, 2).reshape(N, -1)], 1).astype(np.float64)
    at = host(ordered)[:, 3].copy().view(np.uint32) if by_position else np.arange(N)
    ref, bound = oracle.encode_fwd(ref_grid, table, u)[at], oracle.encode_fwd(ref_grid, table, u, abs_terms=True)[at]
    assert np.all(np.abs(got - ref) <= 2.0 ** -11 * np.abs(ref) + 1e-5 * bound + 6e-8)          # as in test_ordered_encode


@pytest.mark.parametrize("name", ["c2_ngp", "c3_2x2", "c8_app"])
def test_step_with_split_features(name, monkeypatch):
    """The training step in spatial order with split features, through every comparison of the plain step; what a caller reads as
    step.feat is planes."""
    from test_gpu_step import _compare_step
    print("[case] step with split features", name, flush=True)
    monkeypatch.setattr(TrainStep, "_order_min", lambda self, m: 1)
    split = []
    monkeypatch.setattr(TrainStep, "_split", lambda self, m, N, use: split.append(N) or True)
    cfg = di.config(name)
    cfg["grid"] = dict(cfg["grid"], log2_T=16)
    _compare_step(cfg, 700, seed=2, lambda1=1e-3, loss_scale=2.0 ** 14, use_jitter_array=False, table_gain=3000.0)
    assert split


def test_refresh_with_split_features(monkeypatch):
    """The refresh of an occupancy grid from split features: the bits of the one from rows, and the candidates' planes for a caller."""
    from test_gpu_step_state import _marched
    print("[case] refresh with split features", flush=True)
    monkeypatch.setattr(TrainStep, "_order_min", lambda self, m: 1)
    seen = []
    for split in (False, True):
        monkeypatch.setattr(TrainStep, "_split", lambda self, m, N, use: split)
        step = _marched()[0]
        assert step.refresh_occupancy(4096) and step._feat_rows[0].levels == (B.SPLIT_LEVELS if split else 16)
        k = min(step.max_samples, step.occ[0].desc.n_cells // 2)
        seen.append((step.occ[0].density.clone(), step.feat[:k].clone()))
    for a, b in zip(*seen):
        assert torch.equal(a, b)


def test_density_of_a_nan_candidate():
    """A NaN among the features: the clip makes the network's NaN -15, the same density as by the separate entry points."""
    print("[case] density of a NaN candidate", flush=True)
    N, n_cells = 40, 40
    mlp = B.dg_mlp_desc(32, 64, 16, 16, 64, 2, 1)
    weights = dev((np.random.default_rng(43).standard_normal(9408) * 0.2).astype(np.float16))
    planes = torch.randn(16, N, 2, device=DEV).half()
    planes[3, 7, 1] = planes[0, 39, 0] = float("nan")
    cell = torch.arange(N, dtype=torch.int32, device=DEV)
    sigma, rgb = torch.zeros(N, device=DEV), torch.zeros(N, 3, device=DEV)
    B.dg_mlp_fwd(mlp, weights, planes, torch.zeros(1, 16, dtype=torch.float16, device=DEV), N, N, sigma, rgb)
    want, got = torch.zeros(n_cells, device=DEV), torch.zeros(n_cells, device=DEV)
    B.dg_occ_update(want, cell, sigma, N)
    B.dg_occ_evaluate(mlp, weights, planes, False, cell, 1, N, got)
    assert torch.equal(got, want) and bool((got > 0).all())
