"""Linears on both sides of the lines between 128- and 64-wide tiles: whole rounds
over the 256 CUs, a second round of one row of tiles, and the last and first grids
around 0.8 of two rounds, against the FP64 oracle with the layer kinds' FP32
tolerance."""
import pytest

torch = pytest.importorskip("torch")

from oracle import gclayers as gcl
from paper_2207_11333_amd import hgnn, synth
from test_gpu_gclayers import rel

pytestmark = pytest.mark.gpu


# H = 256: two columns of 128-wide tiles, 256, 258, 408 and 410 of them
@pytest.mark.parametrize("nodes", [128 * 128, 128 * 128 + 1, 204 * 128, 204 * 128 + 1])
def test_rounds(nodes):
    n = nodes % 32
    b = synth.make_batch(91, nodes // 32 - 1, 32, 32, 1)
    b = synth.concat_batches([b, synth.make_batch(92, 1, 32 + n, 32 + n, 1)])
    assert b.num_nodes == nodes
    params = synth.init_gc_params("sage", 2, 256, 93, edge_feat=1)
    m = hgnn.Model(2, 256, 9, 1, 4, 0, 0, 1.0, kind="sage")
    m.set_params(params)
    pred = torch.empty(b.num_graphs, device="cuda")
    m.forward(hgnn.DeviceBatch.from_host(b), pred)
    rec = gcl.forward(params, b, "sage", 2, 256)
    assert rel(pred.cpu().numpy(), rec.y[:, 0]) <= 1e-5
    m.close()
