"""Small batches in a context that has seen a large one: their backward pass forms
the weight gradients in one launch as in a fresh context, adds the buffers for that
at its first such pass, and does without them under stream capture or where their
allocation fails.  The gradients are the same bits on every route."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2207_11333_amd import synth

pytestmark = pytest.mark.gpu

L, H = 3, 64


def _hg():
    from paper_2207_11333_amd import hgnn
    return hgnn


def _model(kind, prec):
    m = _hg().Model(L, H, 9, 1, 4, prec, 0, 1.08, kind=kind)
    m.set_params(synth.init_params(synth.ModelShape(L, H, 9, 1), 23) if kind == "pna"
                 else synth.init_gc_params(kind, L, H, 23))
    return m


class _Step:
    def __init__(self, m, b):
        self.m, self.db = m, _hg().DeviceBatch.from_host(b)
        self.pred = torch.empty(b.num_graphs, device="cuda")
        self.loss = torch.empty(1, device="cuda")

    def __call__(self):
        self.m.forward(self.db, self.pred, self.loss)
        self.m.backward()

    def grads(self):
        self()
        return self.m.grads()


def _launches(m, step):
    """Weight-gradient launches of a pass (every product, or all in one)."""
    n = 0
    for site in ("update_wgrad", "message_wgrad"):
        m.timer_start(site, 64)
        step()
        n += m.timer_read()[1]
    return n


def _batches():
    small = synth.make_batch(21, 30, 10, 60, 1)
    large = synth.concat_batches([synth.make_batch(22, 64, 60, 70, 1)] * 4)
    assert large.num_nodes >= 16384 > small.num_nodes
    return small, large


KINDS = [(k, p) for k in ("pna", "sage", "cgcnn") for p in (0, 1)]


@pytest.mark.parametrize("kind,prec", KINDS)
def test_small_batch_after_a_large_one(kind, prec):
    small, large = _batches()
    fresh = _model(kind, prec)
    want = _Step(fresh, small).grads()
    m = _model(kind, prec)
    sm, la = _Step(m, small), _Step(m, large)
    big = la.grads()
    assert torch.equal(sm.grads(), want)
    assert _launches(m, sm) == 1 and _launches(m, la) >= L
    assert torch.equal(la.grads(), big)
    assert torch.equal(sm.grads(), want)
    m.close()
    fresh.close()


@pytest.mark.parametrize("kind,prec", KINDS)
def test_captured_before_any_eager_pass(kind, prec):
    """The first small pass of a grown context is recorded: no allocation then."""
    small, large = _batches()
    m = _model(kind, prec)
    sm, la = _Step(m, small), _Step(m, large)
    big = la.grads()
    m.forward(sm.db, sm.pred, sm.loss)  # weights staged, no backward
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        sm()
    want = _Step(_model(kind, prec), small).grads()
    for _ in range(3):
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(m.grads(), want)
        assert torch.equal(la.grads(), big)
        assert torch.equal(sm.grads(), want)
    m.close()


# a small context's first workspace, and the buffers added to a grown one
@pytest.mark.parametrize("grown", [False, True])
@pytest.mark.parametrize("kind,prec", KINDS)
def test_without_memory_for_the_one_launch(kind, prec, grown):
    small, large = _batches()
    want = _Step(_model(kind, prec), small).grads()
    for n in (1, 2, 3, 4, 30):
        m = _model(kind, prec)
        sm = _Step(m, small)
        if grown:
            big = _Step(m, large).grads()
        m.debug_fail_alloc(n)
        assert torch.equal(sm.grads(), want)
        m.debug_fail_alloc(0)
        buffers = 5 if kind == "pna" else 3  # of the one launch; a workspace has over 30
        assert (_launches(m, sm) == 1) == (grown and n > buffers)
        if grown:
            assert torch.equal(_Step(m, large).grads(), big)
        assert torch.equal(sm.grads(), want)
        m.check()
        m.close()
