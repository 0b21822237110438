"""What a step keeps between its calls: a second backward pass on one forward pass, the feature buffers as other calls
leave them, tensors of the caller's own in place of the step's."""
import pytest
import torch

import dg_inputs as di
import oracle.step as ostep
from gpu_util import TOL_F16, TOL_F32, dev, gpu_models, gpu_occupancy, have_gpu, host, make_step, rel_err
from paper_2405_04416_amd import binding as B
from paper_2405_04416_amd.step import TrainStep

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not have_gpu(), reason="needs a GPU")]

R = 301


@pytest.fixture
def ordered(monkeypatch):
    """Samples in spatial order from the first sample on."""
    monkeypatch.setattr(TrainStep, "_order_min", lambda self, m: 1)


def _step(seed=4, loss_scale=2.0 ** 14, **kw):
    cfg = di.config("c2_ngp")
    cfg["table_range"] *= 3000.0
    o, d = di.make_rays(cfg, seed=seed, R=R)
    models = gpu_models(cfg, ostep.make_models(cfg, seed=seed))
    step = make_step(cfg, models, R, loss_scale=loss_scale, lambda1=1e-3, seed=seed, **kw)
    return step, models[0], dev(o), dev(d), dev(di.make_targets(R, seed=seed))


def test_backward_after_an_overflow(ordered):
    """Deltas that overflow fp16 spoil that pass alone: with a smaller loss scale, the next backward pass on the same
    forward pass gives the gradients of a step that never overflowed."""
    print("[case] backward after an overflow", flush=True)
    step, m, o, d, target = _step()
    step.step(o, d, target)
    want, want_w = host(m.dtable), host(m.dW)
    assert step.layout[0][2] is not None
    step.loss_scale = 2.0 ** 60
    step.backward()
    assert not bool(torch.isfinite(m.dW).all()) and not bool(torch.isfinite(m.dtable).all())
    step.loss_scale = 2.0 ** 14
    step.backward()
    # the same arithmetic in another order of the atomic adds
    assert rel_err(host(m.dtable), want) <= TOL_F32 and rel_err(host(m.dW), want_w) <= TOL_F32


def test_backward_with_smaller_seeds(ordered):
    """Seeds 2^-30 times as large (and a loss scale 2^30 times as large, so that the deltas are the same) give gradients
    2^-30 times as large, whatever an earlier backward pass saw."""
    print("[case] backward with smaller seeds", flush=True)
    step, m, o, d, target = _step()
    step.step(o, d, target)
    want = host(m.dtable) * 2.0 ** -30
    step.gC.mul_(2.0 ** -30)
    step.gT.mul_(2.0 ** -30)
    step.loss_scale *= 2.0 ** 30
    step.backward()
    assert rel_err(host(m.dtable), want) <= TOL_F32


def test_feature_buffers_after_other_calls(ordered):
    """Rendering other rays rewrites the features and leaves the feature gradient of the last backward pass alone."""
    print("[case] feature buffers after a rendering", flush=True)
    step, m, o, d, target = _step()
    step.step(o, d, target)
    n = step.layout[0][1]
    want = step.dfeat.clone()
    step.step(o, d, target)                         # the gradient lies in rows again
    _, _, o2, d2, _ = _step(seed=9)
    step.render(o2, d2)
    assert step.layout[0][1] != n
    assert rel_err(host(step.dfeat[:n]), host(want[:n])) <= 1e-6
    k = step.layout[0][1]
    plain = torch.zeros(k, 32, dtype=torch.float16, device=want.device)
    B.dg_hashgrid_encode_fwd(m.grid, m.table, step.u[:k], k, plain)
    # the two encodes add a cell's corners up in another order before the rounding to fp16
    assert rel_err(host(step.feat[:k]), host(plain)) <= 2.0 ** -10


def test_feature_buffers_are_live(ordered):
    """feat and dfeat are the step's own buffers: what a caller writes or puts there between the forward and the backward
    pass is what the backward pass takes, and both can be replaced."""
    print("[case] feature buffers are live", flush=True)
    step, m, o, d, target = _step()
    step.step(o, d, target)
    want, want_w = host(m.dtable), host(m.dW)
    step.forward(o, d, target)
    n = step.layout[0][1]
    feat = step.feat
    step.backward()                                 # read, not changed: the same gradients, by the plain kernels
    assert rel_err(host(m.dtable), want) <= TOL_F16 and rel_err(host(m.dW), want_w) <= TOL_F16
    dfeat = step.dfeat
    assert feat.data_ptr() == step.feat.data_ptr() and dfeat.data_ptr() == step.dfeat.data_ptr()
    step.forward(o, d, target)
    step.feat[:n].zero_()
    step.backward()
    assert float(m.dW[:64 * 32].abs().max()) == 0.0             # the first layer saw no input
    mine, mine_g = torch.zeros_like(feat), torch.zeros_like(dfeat)
    step.feat, step.dfeat = mine, mine_g
    step.step(o, d, target)
    assert step.feat is mine and step.dfeat is mine_g
    assert rel_err(host(m.dtable), want) <= TOL_F32 and float(mine.abs().max()) > 0 and float(mine_g.abs().max()) > 0


@pytest.mark.parametrize("which", ["loss", "status", "both"])
def test_words_of_the_caller(which):
    """loss and status can be tensors of the caller's own: they are cleared at the start of a step as the step's are."""
    print("[case] words of the caller", which, flush=True)
    step, m, o, d, target = _step()
    step.step(o, d, target)
    want = float(step.loss)
    if which != "status":
        step.loss = torch.full((1,), 5.0, device=step.dev)
    if which != "loss":
        step.status = torch.full((1,), 7, dtype=torch.int32, device=step.dev)
    for _ in range(2):
        step.step(o, d, target)
        assert float(step.loss) == pytest.approx(want, rel=TOL_F32) and int(step.status) == 0


def _marched(seed=7):
    cfg = di.config("c7_occ")
    cfg["table_range"] *= 3000.0
    cfg["occ"] = dict(cfg["occ"], res=32)
    o, d = di.make_rays(cfg, seed=seed, R=R)
    models = gpu_models(cfg, ostep.make_models(cfg, seed=seed))
    q = gpu_occupancy(cfg, ostep.make_occupancy(cfg, seed=seed))
    step = make_step(cfg, models, R, loss_scale=2.0 ** 14, seed=seed, occupancy=q, max_samples=1 << 16)
    return step, models[0], dev(o), dev(d), dev(di.make_targets(R, seed=seed))


def test_feature_buffers_after_a_refresh(ordered):
    """The occupancy refresh uses the feature buffer as scratch, in sorted order; what is read afterwards is in the order of its
    candidates.  The gradient buffer is not touched, and a backward pass after it runs on planes."""
    print("[case] feature buffers after a refresh", flush=True)
    step, m, o, d, target = _marched()
    step.step(o, d, target)
    assert step.layout[0][2] is not None
    n = step.layout[0][1]
    want = step.dfeat.clone()
    step.step(o, d, target)
    assert step.refresh_occupancy(4096)
    assert rel_err(host(step.dfeat[:n]), host(want[:n])) <= 1e-6
    k = min(step.max_samples, step.occ[0].desc.n_cells // 2)
    plain = torch.zeros(k, 32, dtype=torch.float16, device=want.device)
    B.dg_hashgrid_encode_fwd(m.grid, m.table, step.u[:k], k, plain)
    assert rel_err(host(step.feat[:k]), host(plain)) <= 2.0 ** -10
    step.forward(o, d, target)
    step.refresh_occupancy(4112)                    # scratch now: the gradients that follow mean nothing, but they are of this step
    step.backward()
    torch.cuda.synchronize()
    assert bool(torch.isfinite(m.dW).all())


@pytest.mark.parametrize("name,R", [("c1_tiny", 257), ("c2_ngp", 1), ("c2_ngp", 700), ("c3_2x2", 500), ("c6_cascade", 300)])
def test_one_call_each_way(name, R, monkeypatch):
    """A sub-model's share of a step in one library call each way and by the single entry points: the same numbers.  The table gradient
    adds up in no fixed order; the caller's own gradient buffers are the ones that are cleared and filled."""
    cfg = di.config(name, table_range=0.3)
    for key in ("grid", "grid_coarse"):
        if key in cfg:
            cfg[key] = dict(cfg[key], log2_T=min(cfg[key]["log2_T"], 16))
    o, d = di.make_rays(cfg, seed=5, R=R)
    target, hm = dev(di.make_targets(R, seed=5)), ostep.make_models(cfg, seed=5)
    steps = [make_step(cfg, gpu_models(cfg, hm), R, seed=5) for _ in range(2)]
    took = []
    one_call = TrainStep._one_call
    for step, allowed in zip(steps, (True, False)):
        monkeypatch.setattr(TrainStep, "_one_call", lambda self, order, N: took.append((allowed, one_call(self, order, N))) or (allowed and took[-1][1]))
        for m in step.models.values():
            m.dtable, m.dW = torch.full_like(m.dtable, 7.0), torch.full_like(m.dW, 7.0)
        for _ in range(2):
            step.step(dev(o), dev(d), target)
    assert all(yes for allowed, yes in took) and any(allowed for allowed, _ in took)
    a, b = steps
    for x, y in ((a.C, b.C), (a.T, b.T), (a.gCk, b.gCk)):
        assert torch.equal(x, y)
    assert float(a.loss) == pytest.approx(float(b.loss), rel=1e-6)
    for p in a.models:
        assert float((a.models[p].dW - b.models[p].dW).norm()) <= 1e-6 * float(b.models[p].dW.norm())
        assert float((a.models[p].dtable - b.models[p].dtable).norm()) <= 1e-6 * float(b.models[p].dtable.norm())


def test_one_call_refuses_buffers_that_are_too_small():
    cfg = di.config("c1_tiny")
    R = 64
    o, d = di.make_rays(cfg, seed=6, R=R)
    step = make_step(cfg, gpu_models(cfg, ostep.make_models(cfg, seed=6)), R, seed=6)
    step.feat = step.feat[:5]
    with pytest.raises(B.DistGridError):
        step.step(dev(o), dev(d), dev(di.make_targets(R, seed=6)))
