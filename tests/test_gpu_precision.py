"""How far a training step's colours, transmittances, loss and weight gradients are from the oracle's, whose sums are in
double precision: bounds in 2-norm per kind of output, four times the largest measured on MI355X over three seeds of each of these
configurations -- colours 6.7e-7, transmittances 3.4e-7, loss 1.1e-7, weight gradients 2.7e-6 (single samples whose hidden unit crosses
a ReLU kink; 1.1e-7 without one).  A sum held in 16 bits anywhere would show as 1e-4."""
import numpy as np
import pytest

import dg_inputs as di
from gpu_util import have_gpu, host, split_appearance_weights
from paper_2405_04416_amd.step import TrainStep

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not have_gpu(), reason="needs a GPU")]


def _off(got, want):
    want = np.asarray(want, np.float64)
    return float(np.linalg.norm(np.asarray(got, np.float64) - want) / np.linalg.norm(want))


# the small grids of c1 are not put in spatial order
@pytest.mark.parametrize("name,R,ordered", [("c1_tiny", 1024, False)] + [(name, R, ordered) for name, R in (("c2_ngp", 1500), ("c3_2x2", 1200), ("c8_app", 1500))
                                                                         for ordered in (False, True)])
def test_step_against_double_precision(name, R, ordered, monkeypatch):
    from test_gpu_step import _compare_step
    print("[case] precision", name, "in spatial order" if ordered else "in ray order", flush=True)
    cfg = di.config(name)
    if ordered:
        monkeypatch.setattr(TrainStep, "_order_min", lambda self, m: 1)
    if name == "c3_2x2":
        cfg["grid"] = dict(cfg["grid"], log2_T=16)
    small = name == "c1_tiny"
    step, ref = _compare_step(cfg, R, seed=1, lambda1=1e-3, loss_scale=4096.0 if small else 2.0 ** 14, use_jitter_array=False,
                              table_gain=1.0 if small else 3000.0)
    assert _off(host(step.C), ref["C"]) <= 2.7e-6
    assert _off(host(step.T), ref["T"]) <= 1.4e-6
    assert abs(float(step.loss) / ref["loss"] - 1.0) <= 4.4e-7
    for p, q in ref["per"].items():
        assert _off(host(step.models[p].dW), split_appearance_weights(q["dW"], q["feat"].shape[1], cfg["mlp"])) <= 1.1e-5, p
