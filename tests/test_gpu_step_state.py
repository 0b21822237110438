"""What a step keeps between its calls: a second backward pass on one forward pass, the feature buffers as other calls
leave them, tensors of the caller's own in place of the step's."""
import numpy as np
import pytest
import torch

import dg_inputs as di
import oracle.step as ostep
from gpu_util import TOL_F32, dev, gpu_models, have_gpu, make_step, rel_err, host
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
