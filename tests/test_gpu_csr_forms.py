"""The one-launch CSR build against the chain of kernels: an edge list off the
16-byte grid takes the chain, whatever the size, and everything that a training
step makes of the two builds (degree-bucket order, edge attributes, scalers and the
padded input among it) is equal bit for bit.  And which faults a malformed
graph_ptr is reported as."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2207_11333_amd import synth
from test_gpu_csr import _batch

pytestmark = pytest.mark.gpu


def _hg():
    from paper_2207_11333_amd import hgnn
    return hgnn


# one workgroup (up to 1024 edges) and several; own nodes in one pass over the
# workgroup's 256 or 1024 threads and in several (many single atoms; graphs of
# more than 1024 atoms), the last one partly filled; a graph per workgroup edge
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("N,E,Fe,maxd,per", [
    (29, 60, 1, 4, 29), (255, 512, 2, 4, 7), (256, 300, 1, 15, 1), (700, 1000, 0, 4, 30),
    (3000, 500, 1, 4, 1), (6144, 1024, 1, 6, 2), (2049, 4096, 1, 15, 2049), (5000, 9000, 3, 4, 2500),
    (6144, 12288, 1, 4, 1030), (4500, 9300, 1, 4, 35)])
def test_one_launch_equals_the_chain(prec, N, E, Fe, maxd, per):
    hg = _hg()
    b = _batch(N + E, N, E, Fe, per, min(maxd, 12))
    H, L, B = 64, 2, b.num_graphs
    m = hg.Model(L, H, 9, Fe, maxd, prec, 0, 1.0)
    m.set_params(synth.init_params(synth.ModelShape(L, H, 9, Fe), 5))
    got = []
    for off in (0, 1):
        db = hg.DeviceBatch.from_host(b)
        ei = torch.empty(2 * E + off, dtype=torch.int32, device="cuda")[off:].view(2, E)
        db.edge_index = ei.copy_(db.edge_index)
        assert (ei.data_ptr() % 16 == 0) == (off == 0)
        pred, loss = torch.empty(B, device="cuda"), torch.empty(1, device="cuda")
        m.forward(db, pred, loss, validate=True)
        m.backward()
        got.append([pred, loss, m.grads()] + [m.fetch(7, l, (N, 4 * H), torch.float32) for l in range(L)]
                   + [m.fetch(8, l, (N, 2 * H), torch.uint8) for l in range(L)]
                   + [m.fetch(i, 0, (n,)) for i, n in ((0, N + 1), (1, E), (2, E), (3, N), (4, N + 1),
                                                       (5, E), (6, N))])
    assert torch.isfinite(got[0][2]).all() and float(got[0][2].abs().max()) > 0
    for k, (a, c) in enumerate(zip(*got)):
        assert torch.equal(a, c), k
    m.close()


@pytest.mark.parametrize("N,E", [(60, 100), (1500, 3000), (6000, 12000)])
def test_malformed_graph_ptr_is_named_alone(N, E):
    hg = _hg()
    b = _batch(N, N, E, 1)
    m = hg.Model(1, 16, 9, 1, 4, 0, 0, 1.0)
    for at, v in ((1, b.graph_ptr[2]), (0, 1), (-1, N - 1)):
        gp = b.graph_ptr.copy()
        gp[at] = v
        bad = synth.Batch(gp, b.x, b.edge_index, b.edge_attr, b.y)
        with pytest.raises(Exception) as e:
            m.prepare(hg.DeviceBatch.from_host(bad), validate=True)
        assert "graph_ptr" in str(e.value) and "crosses" not in str(e.value)
    m.close()
