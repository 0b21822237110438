"""GPU parity of the whole forward + backward pass with occupancy-guided sampling (Sec. 3.2, Sec. 5.1), and of the
occupancy refresh, against the oracle.  Sample bookkeeping is bit-exact; values follow the bars of the fixed-sample
step (fp16 MLP, atomically accumulated gradients: 2e-3)."""
import sys

import numpy as np
import pytest
import torch

import dg_inputs as di
import oracle
import oracle.step as ostep

from gpu_util import (DEV, TOL_F16, TOL_F32, assert_close_robust, dev, from_planes, gpu_models, gpu_occupancy, have_gpu, host,
                      make_step, rel_err, split_appearance_weights)
from paper_2405_04416_amd import binding as B
from paper_2405_04416_amd.step import TrainStep

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not have_gpu(), reason="needs a GPU")]


def say(msg):
    print("[case]", msg)
    sys.stdout.flush()


def _compare(cfg, R, seed, lambda1, loss_scale, table_gain, max_samples):
    cfg = dict(cfg)
    cfg["table_range"] = cfg["table_range"] * table_gain
    o, d = di.make_rays(cfg, seed=seed, R=R)
    Cgt = di.make_targets(R, seed=seed)
    hm = ostep.make_models(cfg, seed=seed)
    ho = ostep.make_occupancy(cfg, seed=seed)
    gm = gpu_models(cfg, hm)
    app_h = app_d = None
    if cfg["mlp"].get("n_app"):
        table, image = di.make_appearance(cfg["n_images"], cfg["mlp"]["n_app"], R, seed=seed)
        app_h, app_d = (table, image), (dev(table), dev(image.view(np.int32)))
    step = make_step(cfg, gm, R, loss_scale=loss_scale, lambda1=lambda1, seed=seed, occupancy=gpu_occupancy(cfg, ho),
                     max_samples=max_samples, appearance=app_d)
    step.step(dev(o), dev(d), dev(Cgt))
    D = step.depth()
    torch.cuda.synchronize()
    ref = ostep.run_step(cfg, hm, o, d, Cgt, seed=seed, lambda1=lambda1, loss_scale=loss_scale, occ=ho, appearance=app_h)
    assert int(host(step.status)[0]) == 0
    np.testing.assert_array_equal(host(step.seg_count), ref["seg_count"])
    np.testing.assert_array_equal(host(step.part_offset), ref["part_offset"])
    for p, q in ref["per"].items():
        b, e = q["b"], q["e"]
        s0, N = step.samples[p]
        assert N == q["u"].shape[0]
        np.testing.assert_array_equal(host(step.first[b + p:e + p + 1]).view(np.uint32), q["first"])
        sl = slice(s0, s0 + N)
        np.testing.assert_array_equal(host(step.u[sl]).view(np.uint32), q["u"].view(np.uint32))
        np.testing.assert_array_equal(host(step.delta[sl]).view(np.uint32), q["delta"].view(np.uint32))
        assert rel_err(from_planes(step.feat[sl], N, q["feat"].shape[1]).astype(np.float64), q["feat"]) <= 1e-3
        assert_close_robust(host(step.sigma[sl]), q["sigma"], TOL_F16, "sigma")
        assert_close_robust(host(step.rgb[sl]), q["rgb"], TOL_F16, "rgb")
    cnt = ref["seg_count"]
    used = np.arange(cfg["k_max"])[None, :] < cnt[:, None]
    assert rel_err(host(step.Ck)[used], ref["Ck"][used]) <= TOL_F16
    assert rel_err(host(step.Tk)[used], ref["Tk"][used]) <= TOL_F16
    assert rel_err(host(step.C), ref["C"]) <= TOL_F16
    assert rel_err(host(step.T), ref["T"]) <= TOL_F16
    assert abs(float(step.loss.item()) - ref["loss"]) <= TOL_F16 * abs(ref["loss"])
    assert rel_err(host(step.gCk)[used], ref["gCk"][used]) <= TOL_F16
    for p, q in ref["per"].items():
        s0, N = step.samples[p]
        sl = slice(s0, s0 + N)
        assert_close_robust(host(step.dsigma[sl]), q["dsigma"], TOL_F16, "dsigma")
        assert_close_robust(host(step.drgb[sl]), q["drgb"], TOL_F16, "drgb")
        assert_close_robust(from_planes(step.dfeat[sl], N, q["dfeat"].shape[1]), q["dfeat"], TOL_F16, "dfeat")
        assert_close_robust(host(gm[p].dW), split_appearance_weights(q["dW"], q["feat"].shape[1], cfg["mlp"]), TOL_F16, "dW")
        grid = hm[p]["grid"]
        got = host(gm[p].dtable).astype(np.float64)
        for l in range(grid.L):
            s2 = slice(grid.first[l], grid.first[l + 1])
            assert_close_robust(got[s2], q["dtable"][s2], TOL_F16, "dtable level %d of part %d" % (l, p), min_outliers=32)
    # depth of the same samples: merged expected distance (Sec. 4.4.2)
    Dk = np.zeros((R, cfg["k_max"]))
    for p, q in ref["per"].items():
        b, e = q["b"], q["e"]
        first, u, delta, t, ray = oracle.march_segments(o, d, ref["seg_t"], ref["seg_ray"], ref["seg_slot"], b, e, cfg["parts"][p],
                                                        ho[p]["grid"], ho[p]["bits"], ho[p]["dt"], ho[p]["max_steps"], seed=seed)
        Dk[ref["seg_ray"][b:e], ref["seg_slot"][b:e]] = oracle.composite_depth_ragged(q["sigma"], delta, t, first)
    refD = oracle.merge_depth(Dk, ref["Tk"], cnt)
    assert rel_err(host(D), refD) <= TOL_F16
    return step, ref


def test_step_occupancy_single_box():
    say("step c7_occ: 1200 rays, occupancy grid of resolution 64, marching step of Instant-NGP")
    cfg = di.config("c7_occ")
    cfg["occ"] = dict(cfg["occ"], res=64)
    step, ref = _compare(cfg, 1200, seed=1, lambda1=1e-3, loss_scale=2.0 ** 14, table_gain=3000.0, max_samples=60000)
    counts = np.diff(ref["per"][0]["first"].astype(np.int64))
    assert counts.max() > 10 and np.any(counts == 0) and 3 < counts.mean() < 60


def test_step_occupancy_four_boxes():
    say("step c3_2x2 with occupancy grids of resolution 48, 900 rays, T = 2^16")
    cfg = di.config("c3_2x2")
    cfg["grid"] = dict(cfg["grid"], log2_T=16)
    cfg["occ"] = dict(res=48, max_steps=512)
    step, ref = _compare(cfg, 900, seed=2, lambda1=1e-3, loss_scale=2.0 ** 14, table_gain=3000.0, max_samples=200000)
    assert len(ref["per"]) == 4


def test_step_occupancy_with_appearance_features():
    say("step c8_app with an occupancy grid of resolution 64: one appearance row per sample, 16 appearance inputs")
    cfg = di.config("c8_app")
    cfg["mlp"] = dict(cfg["mlp"], n_app=16)
    cfg["occ"] = dict(res=64, max_steps=1024)
    _compare(cfg, 1000, seed=4, lambda1=1e-3, loss_scale=2.0 ** 14, table_gain=3000.0, max_samples=60000)


@pytest.mark.parametrize("full,factor", [(False, 3.0), (True, 1.5)])
def test_bricks_of_guided_samples(monkeypatch, full, factor):
    """Samples on surfaces are put in bricks for three times their number; those of a grid that is set all over fill the box and are not.  Where the
    workspace is too small for the levels that are then left unmerged, the bricks are those of samples on surfaces."""
    say("bricks of occupancy-guided samples, grid full: %s" % full)
    monkeypatch.setattr(TrainStep, "_order_min", lambda self, m: 1)
    cfg = di.config("c7_occ")
    cfg["grid"] = dict(cfg["grid"], log2_T=18)
    cfg["occ"] = dict(cfg["occ"], res=64)
    R = 20000
    o, d = di.make_rays(cfg, seed=5, R=R)
    hm, ho = ostep.make_models(cfg, seed=5), ostep.make_occupancy(cfg, seed=5)
    if full:
        ho[0]["bits"] = ~np.zeros_like(ho[0]["bits"])
    gm = gpu_models(cfg, hm)
    step = make_step(cfg, gm, R, loss_scale=2.0 ** 14, seed=5, occupancy=gpu_occupancy(cfg, ho), max_samples=100 * R)
    step.step(dev(o), dev(d), dev(di.make_targets(R, seed=5)))
    N = step.samples[0][1]
    assert N > (50 if full else 3) * R // 2
    assert bytes(step.layout[0][2]) == bytes(B.dg_order_desc_init(gm[0].grid, int(factor * N)))
    if full:
        step.ws_enc = step.ws_enc[:B.dg_hashgrid_encode_bwd_ordered_workspace_bytes(gm[0].grid, step.layout[0][2], N) // 4 - 64]
        step.step(dev(o), dev(d), dev(di.make_targets(R, seed=5)))
        assert bytes(step.layout[0][2]) == bytes(B.dg_order_desc_init(gm[0].grid, 3 * N))
    torch.cuda.synchronize()
    assert bool(torch.isfinite(gm[0].dtable).all()) and bool(gm[0].dtable.any())


def test_sample_capacity_is_enforced():
    say("step c7_occ: too little room for the samples raises")
    cfg = di.config("c7_occ")
    cfg["occ"] = dict(cfg["occ"], res=64)
    R = 500
    o, d = di.make_rays(cfg, seed=1, R=R)
    hm = ostep.make_models(cfg, seed=1)
    ho = ostep.make_occupancy(cfg, seed=1)
    step = make_step(cfg, gpu_models(cfg, hm), R, occupancy=gpu_occupancy(cfg, ho), max_samples=100)
    from paper_2405_04416_amd.binding import DistGridError
    with pytest.raises(DistGridError):
        step.forward(dev(o), dev(d), dev(di.make_targets(R, seed=1)))
    torch.cuda.synchronize()
    assert int(host(step.status)[0]) == 2


@pytest.mark.parametrize("iteration", [0, 16, 4112, 10000, 7])
def test_occupancy_refresh(iteration):
    say("occupancy refresh at iteration %d" % iteration)
    cfg = di.config("c7_occ")
    cfg["occ"] = dict(cfg["occ"], res=40)
    cfg["table_range"] = 5.0                                        # the field's densities spread over 0.2 .. 20
    hm = ostep.make_models(cfg, seed=3)
    ho = ostep.make_occupancy(cfg, seed=3)
    for q in ho.values():                                          # stand-in densities on the scale of this field's
        q["density"] = (q["density"] * 0.02).astype(np.float32)
    step = make_step(cfg, gpu_models(cfg, hm), 64, occupancy=gpu_occupancy(cfg, ho), max_samples=3000)   # several pieces
    before = host(step.occ[0].density).copy()
    did = step.refresh_occupancy(iteration)
    torch.cuda.synchronize()
    assert did == ostep.refresh_occupancy(hm, ho, iteration, seed=0)
    assert did == (iteration % 16 == 0)
    if not did:
        np.testing.assert_array_equal(host(step.occ[0].density), before)
        return
    q = ho[0]
    got = host(step.occ[0].density)
    assert_close_robust(got, q["density"], TOL_F16, "density")
    thr = oracle.occ_schedule(iteration)[3]
    clear = np.abs(q["density"] - thr) > 4 * TOL_F16 * thr          # cells whose bit the fp16 field cannot flip
    gb = np.unpackbits(host(step.occ[0].bits).view(np.uint8), bitorder="little")[:got.size].astype(bool)
    rb = np.unpackbits(q["bits"].view(np.uint8), bitorder="little")[:got.size].astype(bool)
    np.testing.assert_array_equal(gb[clear], rb[clear])
    np.testing.assert_array_equal(gb, got > np.float32(thr))        # the bits belong to the library's own densities
    assert int(host(step.occ[0].n_set)[0]) == int(gb.sum())
    assert 0 < q["last_sigma"].min() and np.unique(q["last_cell"]).size > 0.3 * q["last_cell"].size


def test_step_occupancy_full_size_bench_configuration():
    """c7_occ at the size and launch configuration bench.py times (2^18 rays, occupancy grid 512 x 512 x 64): rays
    sampled from the batch through the oracle one by one, and properties that hold at any size."""
    say("step c7_occ full size (2^18 rays, occupancy resolution 512)")
    from paper_2405_04416_amd import binding as B
    cfg = di.config("c7_occ")
    R = cfg["R"]
    o, d = di.make_rays(cfg, seed=0)
    Cgt = di.make_targets(R, seed=0)
    hm = ostep.make_models(cfg, seed=0)
    hm[0]["table"] *= np.float32(3000.0)
    ho = ostep.make_occupancy(cfg, seed=0)
    gm = gpu_models(cfg, hm)
    step = make_step(cfg, gm, R, loss_scale=2.0 ** 16, lambda1=1e-3, seed=0, occupancy=gpu_occupancy(cfg, ho), max_samples=R * 32)
    step.step(dev(o), dev(d), dev(Cgt))
    torch.cuda.synchronize()
    assert int(host(step.status)[0]) == 0
    n_seg = step.offsets[-1]
    s0, N = step.samples[0]
    first = host(step.first[:n_seg + 1]).astype(np.int64)
    counts = np.diff(first)
    say("segments %d, samples %d (%.2f per segment)" % (n_seg, N, N / n_seg))
    assert s0 == 0 and first[0] == 0 and first[-1] == N and counts.min() >= 0 and 2.0 < N / n_seg < 40.0

    # (a) 64 sampled rays through the oracle, each marched on its own
    cnt = host(step.seg_count)
    pos_of_ray = np.cumsum(cnt) - cnt                       # k_max = 1: bucket order is ray order among hits
    seg_t = host(step.seg_t)
    q, box = ho[0], cfg["parts"][0]
    pick = np.random.default_rng(0).choice(np.nonzero(cnt)[0], 64, replace=False)
    checked = 0
    for r in pick:
        f1, u, delta, t, ray = oracle.march_segments(o, d, seg_t, np.array([r], np.uint32), np.array([0], np.uint32), 0, 1, box,
                                                     q["grid"], q["bits"], q["dt"], q["max_steps"], seed=0)
        j = int(pos_of_ray[r])
        assert counts[j] == f1[1]
        sl = slice(int(first[j]), int(first[j + 1]))
        np.testing.assert_array_equal(host(step.u[sl]).view(np.uint32), u.view(np.uint32))
        np.testing.assert_array_equal(host(step.delta[sl]).view(np.uint32), delta.view(np.uint32))
        if f1[1] == 0:
            assert float(step.T[r]) == 1.0 and np.all(host(step.C[r]) == 0)
            continue
        feat = oracle.encode_fwd(hm[0]["grid"], hm[0]["table"], u)
        sig, rgb = oracle.mlp_fwd(hm[0]["mlp"], hm[0]["weights"].astype(np.float64), feat, oracle.sh(d[ray], 4), 1)
        Cs, Ts = oracle.composite_fwd_ragged(sig, rgb, delta.astype(np.float64), f1)
        assert rel_err(host(step.sigma[sl]), sig) <= TOL_F16
        assert rel_err(host(step.C[r]), Cs[0], floor=1e-3) <= TOL_F16
        assert abs(float(step.T[r]) - Ts[0]) <= TOL_F16
        checked += 1
    assert checked > 30

    # (b) properties that hold at any size
    seg_ray = host(step.seg_ray[:n_seg])
    np.testing.assert_array_equal(host(step.sample_ray[:N]), np.repeat(seg_ray, counts))       # samples are segment-major
    some = np.random.default_rng(1).choice(N, 20000, replace=False)
    cells = oracle.occ_cell(q["grid"], host(step.u[:N])[some])
    assert np.all((q["bits"][cells >> 5] >> (cells & 31)) & 1)                                 # every kept sample is in an occupied cell
    lens = seg_t[seg_ray, 0, 1] - seg_t[seg_ray, 0, 0]
    width = host(step.delta[:N])
    assert np.all(width <= np.float32(q["dt"]) * (1 + 1e-6))                                   # strata no wider than the marching step
    np.testing.assert_allclose(width[first[:-1][counts > 0]], (lens / np.ceil(lens / q["dt"]))[counts > 0], rtol=1e-4)
    m = gm[0]
    L = m.grid.n_levels
    dfeat = step.dfeat[:N].reshape(L, N, 2).double()
    dtab = m.dtable.double()
    probe = torch.rand_like(m.table) - 0.5
    f2 = torch.zeros(L, N, 2, device=DEV)
    B.dg_hashgrid_encode_fwd(m.grid, probe, step.u[:N], N, f2)
    lhs = float((dfeat * f2.double()).sum()); rhs = float((dtab * probe.double()).sum())
    mag = float((dfeat.abs() * f2.double().abs()).sum())
    assert abs(lhs - rhs) <= TOL_F16 * mag                                                     # transpose identity of the encode
    miss = torch.nonzero(step.seg_count == 0).flatten()
    assert bool((step.T[miss] == 1).all()) and bool((step.C[miss] == 0).all())
