"""Weight gradients of a whole backward pass in one launch (small batches)
against the same products launched layer by layer (recomputation, and batches
past the one-launch limit).  Both sum the same chunks in the same order, so
the gradients are equal bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2207_11333_amd import synth

pytestmark = pytest.mark.gpu


def _hg():
    from paper_2207_11333_amd import hgnn
    return hgnn


def _grads(m, b):
    hg = _hg()
    db = hg.DeviceBatch.from_host(b)
    pred = torch.empty(b.num_graphs, device="cuda")
    loss = torch.empty(1, device="cuda")
    m.forward(db, pred, loss)
    m.backward()
    return m.grads().cpu().numpy()


# hidden widths around the 64- and 128-wide output tiles, edge-feature counts
# (rows that keep only their sum column), and batches from a single atom (no
# edge, one node row) over partial 16- and 32-row steps to several chunks
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("H,Fe,graphs,lo,hi", [
    (16, 0, 1, 1, 1), (48, 1, 1, 17, 17), (64, 2, 3, 5, 9), (80, 4, 40, 5, 30),
    (128, 1, 128, 10, 60), (144, 3, 20, 16, 16), (512, 1, 9, 4, 40)])
def test_one_launch_equals_layer_by_layer(prec, H, Fe, graphs, lo, hi):
    b = synth.make_batch(11, graphs, lo, hi, Fe)
    p = synth.init_params(synth.ModelShape(2, H, 9, Fe), 12)
    got = []
    for recompute in (0, 1):
        m = _hg().Model(2, H, 9, Fe, 4, prec, recompute, 1.08)
        m.set_params(p)
        got.append(_grads(m, b))
        m.close()
    assert np.isfinite(got[0]).all() and np.abs(got[0]).max() > 0
    assert np.array_equal(got[0], got[1])


@pytest.mark.parametrize("kind,prec", [("pna", 0), ("pna", 1), ("sage", 0), ("sage", 1),
                                       ("cgcnn", 0), ("cgcnn", 1)])
def test_batches_on_both_sides_of_the_limit(kind, prec):
    small = synth.make_batch(21, 30, 10, 60, 1)
    large = synth.concat_batches([synth.make_batch(22, 64, 60, 70, 1)] * 4)
    assert large.num_nodes >= 16384 > small.num_nodes
    p = (synth.init_params(synth.ModelShape(3, 32, 9, 1), 23) if kind == "pna"
         else synth.init_gc_params(kind, 3, 32, 23))
    got = []
    for order in ((small, large, small), (large, small)):
        m = _hg().Model(3, 32, 9, 1, 4, prec, 0, 1.08, kind=kind)
        m.set_params(p)
        for b in order:
            g = _grads(m, b)
            got.append((b is small, g))
        m.close()
    smalls = [g for s, g in got if s]
    larges = [g for s, g in got if not s]
    assert all(np.array_equal(smalls[0], g) for g in smalls[1:])
    assert np.array_equal(larges[0], larges[1])
