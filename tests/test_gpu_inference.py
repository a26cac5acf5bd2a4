"""Inference workspaces hold the BF16 copies in the room of layer 0's FP32
aggregates and skip what only a backward pass reads; their predictions are the
training forward's, bit for bit.  So are a recomputing context's gradients,
whose forward skips the stored aggregates too."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2207_11333_amd import synth

pytestmark = pytest.mark.gpu


def _hg():
    from paper_2207_11333_amd import hgnn
    return hgnn


# widths with copies (multiples of 64) and without, one layer (no copy is read)
# to five (both rotating outputs), tile edges of the batch (1 node, 64, 65, a
# batch on the 128-wide tiles)
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("H,L,Fe,maxd,graphs,lo,hi", [
    (64, 1, 1, 4, 9, 5, 9), (64, 2, 0, 4, 1, 1, 1), (128, 3, 1, 4, 1, 64, 64),
    (192, 4, 2, 4, 1, 65, 65), (80, 3, 1, 4, 7, 10, 30), (128, 5, 1, 4, 120, 10, 60),
    (128, 3, 1, 20, 30, 10, 60), (256, 2, 4, 6, 140, 30, 60)])
def test_inference_equals_training_forward(prec, H, L, Fe, maxd, graphs, lo, hi):
    b = synth.make_batch(31, graphs, lo, hi, Fe)
    other = synth.make_batch(32, 3, 4, 20, Fe)
    m = _hg().Model(L, H, 9, Fe, maxd, prec, 0, 1.08)
    m.set_params(synth.init_params(synth.ModelShape(L, H, 9, Fe), 33))
    for x in (b, other, b):
        db = _hg().DeviceBatch.from_host(x)
        want = torch.empty(x.num_graphs, device="cuda")
        got = torch.full((x.num_graphs,), np.nan, device="cuda")
        m.forward(db, want)
        m.forward_noalloc(db, got, validate=True)
        assert torch.isfinite(got).all()
        assert torch.equal(want, got)
    m.close()


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("H,L,graphs", [(128, 1, 20), (128, 4, 100), (80, 3, 20), (256, 3, 500)])
def test_recomputation_equals_stored(prec, H, L, graphs):
    b = synth.make_batch(41, graphs, 20, 60, 1)
    p = synth.init_params(synth.ModelShape(L, H, 9, 1), 42)
    got = []
    for recompute in (0, 1):
        m = _hg().Model(L, H, 9, 1, 4, prec, recompute, 1.08)
        m.set_params(p)
        db = _hg().DeviceBatch.from_host(b)
        pred, loss = torch.empty(graphs, device="cuda"), torch.empty(1, device="cuda")
        for _ in range(2):
            m.forward(db, pred, loss)
            m.backward()
        got.append((pred.cpu().numpy(), m.grads().cpu().numpy()))
        m.close()
    assert np.array_equal(got[0][0], got[1][0])
    assert np.array_equal(got[0][1], got[1][1])


# BF16 linears sum in one order whatever tile they run on (128, 64 or 32 a side,
# by the size of the grid), so a graph's prediction does not depend on what else
# is in its batch
@pytest.mark.parametrize("H,graphs,lo,hi", [(128, 700, 58, 62), (128, 300, 50, 60),
                                            (256, 130, 20, 60), (64, 500, 20, 60)])
def test_prediction_independent_of_the_batch(H, graphs, lo, hi):
    b = synth.make_batch(51, graphs, lo, hi, 1)
    m = _hg().Model(3, H, 9, 1, 4, 1, 0, 1.08)
    m.set_params(synth.init_params(synth.ModelShape(3, H, 9, 1), 52))

    def pred(x):
        p = torch.empty(x.num_graphs, device="cuda")
        m.forward(_hg().DeviceBatch.from_host(x), p)
        return p.cpu().numpy()

    whole = pred(b)
    at = 0
    for n in (1, 20, 40, graphs - 61):
        n0, n1 = b.graph_ptr[at], b.graph_ptr[at + n]
        e = (b.edge_index[1] >= n0) & (b.edge_index[1] < n1)
        part = synth.Batch((b.graph_ptr[at:at + n + 1] - n0).astype(np.int32), b.x[n0:n1].copy(),
                           (b.edge_index[:, e] - n0).astype(np.int32), b.edge_attr[e].copy(),
                           b.y[at:at + n].copy())
        assert np.array_equal(pred(part), whole[at:at + n])
        at += n
    m.close()
