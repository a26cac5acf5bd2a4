"""The first layer's linears end their first segment inside a K tile on small
grids.  What lies past the segment there (the next segment's weights, or the
row's first ones) has no part in the sum: an infinite weight reaches the outputs
that its own column gives, and nothing else."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2207_11333_amd import synth

pytestmark = pytest.mark.gpu


def _layer0(F, H, inf_at):
    """Layer 0's outputs and aggregates on 40 nodes, the weight at inf_at(F, H) infinite."""
    from paper_2207_11333_amd import hgnn
    rng = np.random.default_rng(F + H)
    b = synth.make_batch(91, 2, 20, 20, 1)
    x = rng.standard_normal((b.num_nodes, F)).astype(np.float32)
    m = hgnn.Model(1, H, F, 1, 4, 0, 0, 1.0)
    db = hgnn.DeviceBatch(b.graph_ptr, x, b.edge_index, b.edge_attr, b.y)
    w = torch.tensor(synth.init_params(synth.ModelShape(1, H, F, 1), 92))[m.layer_slices()[0]].cuda()
    w[inf_at(F, H)] = float("inf")
    m.prepare(db, validate=True)
    out = hgnn.PNALayerFunction.apply(db.x, w, m, 0)
    A = m.fetch(7, 0, (b.num_nodes, 4 * H), torch.float32)
    deg = m.fetch(3, 0, (b.num_nodes,))
    m.close()
    return torch.tensor(x), out.cpu(), A.cpu(), deg.cpu()


# F pads to 16 and 48 columns: one short K tile, and one after a whole one
@pytest.mark.parametrize("F", [9, 40])
@pytest.mark.parametrize("H", [64, 128])
def test_infinite_weight_past_the_segment(F, H):
    # W^p [H, F + 12H] row 3, the first aggregate column (mean of feature 0), unscaled
    x, out, A, deg = _layer0(F, H, lambda F, H: H * (2 * F + 1) + H + 3 * (F + 12 * H) + F)
    a = A[:, 0]
    assert (a > 0).any() and (a < 0).any()
    assert torch.isinf(out[a > 0, 3]).all()
    assert (out[a < 0, 3] == 0).all()
    assert torch.isfinite(out[:, torch.arange(H) != 3]).all()


@pytest.mark.parametrize("F", [9, 40])
@pytest.mark.parametrize("H", [64, 128])
def test_infinite_weight_in_the_segment(F, H):
    # W^m [H, 2F + 1] row 3, the destination's feature 5: messages of +-infinity
    x, out, A, deg = _layer0(F, H, lambda F, H: 3 * (2 * F + 1) + 5)
    on = deg > 0
    assert on.any()
    assert torch.equal(A[on, 3], torch.sign(x[on, 5]) * float("inf"))
    cols = torch.arange(4 * H) % H != 3
    assert torch.isfinite(A[:, cols]).all()
