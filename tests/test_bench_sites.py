"""The bench's roofline of the weight-gradient sites by how the launches come: a
product each, a layer's two in one launch, every layer's in one."""
import dataclasses
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

torch = pytest.importorskip("torch")


class _Timer:
    """A context whose timed sites have the given launches a step, 10 us each."""

    def __init__(self, per_step, steps):
        self.n = {k: v * steps for k, v in per_step.items()}

    def timer_start(self, site, max_launches):
        self.site = site
        assert max_launches >= self.n.get(site, 0)

    def timer_read(self):
        n = self.n.get(self.site, 0)
        return 0.01 * n, n


@pytest.mark.parametrize("layers", [1, 6])
@pytest.mark.parametrize("recompute,update,message,kernel", [
    (0, "L", "L", "k_wgrad |"), (1, "L", 0, "k_wgrad_pair<0,"), (0, 1, 0, "k_wgrad_all<0,")])
def test_weight_gradient_sites(monkeypatch, layers, recompute, update, message, kernel):
    import bench
    from paper_2207_11333_amd import synth
    monkeypatch.setattr(torch.cuda, "synchronize", lambda: None)
    w = dataclasses.replace(synth.WORKLOADS["c1_train_fp32"], num_layers=layers, recompute=recompute)
    N, E, steps = 4484, 9584, 5
    per = {"update_wgrad": layers if update == "L" else update,
           "message_wgrad": layers if message == "L" else message}
    out = bench.time_sites(_Timer(per, steps), lambda: None, steps, w, N, E)
    upd, _ = bench.site_work("update_wgrad", w, N, E)
    msg, _ = bench.site_work("message_wgrad", w, N, E)
    got = sum(s["flops_per_launch"] * s["launches_per_step"] for s in out.values())
    assert got == pytest.approx(layers * (upd + msg))
    assert out["update_wgrad"]["kernel"].startswith(kernel)
    for name, s in out.items():
        assert s["launches"] == per[name] * steps
        assert s["us_per_step"] == pytest.approx(10 * per[name])
