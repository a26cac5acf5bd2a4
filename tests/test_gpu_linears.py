"""FP32 linears in chunks of K: the LDS-DMA form sums the chunks that split-K
would launch.  Widths and batches that give one chunk, two to four (one running
total), five to eight (two halves), and widths it leaves to the other form,
against the FP64 oracle with the layer kinds' FP32 tolerance."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import gclayers as gcl
from paper_2207_11333_amd import synth
from test_gpu_gclayers import TAU_FP32, _batch, _run, _tensor_report, rel, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,H,B,lo,hi", [
    ("sage", 64, 300, 20, 40),   # one chunk, 64-wide tiles
    ("sage", 128, 1, 1, 1),      # two chunks, one row
    ("sage", 192, 3, 20, 30),    # three
    ("sage", 256, 2, 30, 33),    # four
    ("sage", 320, 2, 31, 33),    # five
    ("sage", 448, 2, 31, 32),    # seven
    ("sage", 512, 4, 15, 17),    # eight
    ("sage", 96, 20, 10, 30),    # not whole 64-deep pieces
    ("cgcnn", 256, 3, 20, 30)])  # with an addend
def test_chunked_sums(kind, H, B, lo, hi):
    b = _batch(61, B, lo, hi, 1)
    params = synth.init_gc_params(kind, 2, H, 62, edge_feat=1)
    m, out = _run(kind, b, params, 2, H, 1)
    rec = gcl.forward(params, b, kind, 2, H)
    g_ref, _ = gcl.backward(rec, out["relu"], out["grelu"], None, tau=TAU_FP32)
    rep = _tensor_report(kind, 2, H, 1, 1, 0, out["grads"], g_ref)
    say(f"{kind} H={H} N={b.num_nodes}: worst gradient {max(rep.values()):.2e}")
    assert rel(out["pred"], rec.y[:, 0]) <= 1e-5
    assert max(rep.values()) <= 1e-5
    m.close()


# BF16 operands rounded in registers (small grids) or while staging (larger ones):
# the same products in the same order, so a graph's prediction does not depend on
# the batch it is in.  2300 to 9300 nodes: both sides of the limit of each linear.
@pytest.mark.parametrize("kind,H,graphs", [("sage", 64, 300), ("sage", 128, 260),
                                           ("cgcnn", 64, 300), ("cgcnn", 128, 200)])
def test_bf16_prediction_independent_of_the_batch(kind, H, graphs):
    from paper_2207_11333_amd import hgnn
    parts = [synth.make_batch(71 + k, n, 30, 32, 1) for k, n in enumerate((1, graphs // 4, graphs))]
    m = hgnn.Model(3, H, 9, 1, 4, 1, 0, 1.0, kind=kind)
    m.set_params(synth.init_gc_params(kind, 3, H, 72, edge_feat=1))

    def pred(b):
        p = torch.empty(b.num_graphs, device="cuda")
        m.forward(hgnn.DeviceBatch.from_host(b), p)
        return p

    whole = pred(synth.concat_batches(parts))
    assert torch.isfinite(whole).all()
    assert torch.equal(torch.cat([pred(b) for b in parts]), whole)
    m.close()


# The first layer's input is padded to 16 columns: K tiles of 16, 32 (none left
# over in FP32), 48 and 64 columns on small grids, the staged form on large ones.
# BF16 sums in one order; FP32 splits K by the size of the batch.
@pytest.mark.parametrize("prec,tol", [(0, 1e-5), (1, 0.0)])
@pytest.mark.parametrize("F", [9, 20, 40, 60])
@pytest.mark.parametrize("H", [64, 128, 80])
def test_first_layer(prec, tol, F, H):
    from paper_2207_11333_amd import hgnn
    rng = np.random.default_rng(F + H)
    parts = []
    for k, n in enumerate((1, 9, 120, 700)):
        b = synth.make_batch(81 + k, n, 12, 16 if n < 700 else 32, 1)
        parts.append(synth.Batch(b.graph_ptr, rng.standard_normal((b.num_nodes, F)).astype(np.float32),
                                 b.edge_index, b.edge_attr, b.y))
    m = hgnn.Model(2, H, F, 1, 4, prec, 0, 1.0)
    m.set_params(synth.init_params(synth.ModelShape(2, H, F, 1), 82))

    def pred(b):
        p = torch.empty(b.num_graphs, device="cuda")
        m.forward(hgnn.DeviceBatch.from_host(b), p)
        return p

    whole = pred(synth.concat_batches(parts))
    got = torch.cat([pred(b) for b in parts])
    assert torch.isfinite(whole).all()
    assert float((got - whole).norm()) <= tol * float(whole.norm())
    m.close()
