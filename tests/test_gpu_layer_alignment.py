"""One layer through the autograd function and the C entries with an input off
the 16-byte grid (a view into a larger buffer, which .contiguous() leaves where
it is): weight gradients of a small layer, whose two products share a launch, and
of a larger one, in both precisions, with and without degree buckets."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2207_11333_amd import synth

pytestmark = pytest.mark.gpu


def _hg():
    from paper_2207_11333_amd import hgnn
    return hgnn


def _rel(a, r):
    return float((a - r).double().norm() / r.double().norm().clamp_min(1e-30))


def _view(t, off):
    """t's values at `off` floats past a 16-byte boundary."""
    v = torch.empty(t.numel() + off, device="cuda")[off:].view(t.shape)
    assert v.is_contiguous() and v.data_ptr() % 16 == 4 * off % 16
    return v.copy_(t)


# H * nodes: 2.6k, 31k and 922k elements (the products of a layer up to 640 * 1024
# run in one launch, above that apart)
@pytest.mark.parametrize("off", [1, 2, 3])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("H,graphs,maxd,recompute", [(64, 1, 4, 0), (48, 20, 4, 0), (256, 100, 4, 0),
                                                     (256, 100, 4, 1), (64, 20, 20, 0)])
def test_layer_input_off_the_grid(off, prec, H, graphs, maxd, recompute):
    hg = _hg()
    b = synth.make_batch(95, graphs, 30, 42, 1)
    N = b.num_nodes
    m = hg.Model(2, H, 9, 1, maxd, prec, recompute, 1.08)
    m.prepare(hg.DeviceBatch.from_host(b), validate=True)
    rng = np.random.default_rng(96)
    t = lambda *s: torch.tensor(rng.standard_normal(s), dtype=torch.float32).cuda()
    h0, g = t(N, H).relu_(), t(N, H)
    w = torch.tensor(synth.init_params(synth.ModelShape(2, H, 9, 1), 97))[m.layer_slices()[1]].cuda()

    # the same stored forward, its backward from the aligned input and from the
    # view: equal bit for bit
    out, dh, dw = torch.empty_like(h0), [], []
    L, p, s = hg.lib(), hg._ptr, hg._stream
    hg._check(L.hgnn_op_layer_forward(m.handle, 1, p(w), p(h0), p(out), s()))
    for h in (h0, _view(h0, off)):
        dh.append(torch.empty_like(h0))
        dw.append(torch.empty_like(w))
        hg._check(L.hgnn_op_layer_backward(m.handle, m.generation(), 1, p(w), p(h), p(out), p(g),
                                           p(dh[-1]), p(dw[-1]), s()))
    assert torch.isfinite(dw[0]).all() and float(dw[0].abs().max()) > 0
    assert torch.equal(dh[0], dh[1])
    assert torch.equal(dw[0], dw[1])

    # the autograd function: the linears take another kernel for such an input, so
    # the outputs are equal but for rounding (FP32 1e-5 a side)
    hv, wv = _view(h0, off).requires_grad_(), w.clone().requires_grad_()
    o = hg.PNALayerFunction.apply(hv, wv, m, 1)
    assert _rel(o.detach(), out) <= (2e-2 if prec else 2e-5)
    a, c = torch.autograd.grad(o, (hv, wv), g)
    assert torch.isfinite(a).all() and torch.isfinite(c).all()
    m.check()
    m.close()
