"""The CSR build at the edges of its size classes (one launch up to 6144 nodes and
12288 edges, of one workgroup up to 1024 edges and of one per 512 above; a chain of
kernels for larger batches) against the host build, and the errors each class
reports."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_2207_11333_amd import synth

pytestmark = pytest.mark.gpu


def _hg():
    from paper_2207_11333_amd import hgnn
    return hgnn


def _batch(seed, N, E, Fe, per=30, cap=4):
    """N nodes in graphs of up to `per`, exactly E directed edges (self-loops and
    repeated pairs among them) of at most `cap` in and out per node, in random order."""
    rng = np.random.default_rng(seed)
    gp = np.append(np.arange(0, N, per), N).astype(np.int32)
    edges, deg = [], np.zeros((2, N), int)
    while len(edges) < E:
        s = int(rng.integers(N))
        g = s // per
        d = int(rng.integers(gp[g], gp[g + 1]))
        if deg[0, s] < cap and deg[1, d] < cap:
            edges.append((s, d))
            deg[0, s] += 1
            deg[1, d] += 1
    ei = np.array(edges, np.int32).reshape(-1, 2).T.copy()
    x = rng.standard_normal((N, 9)).astype(np.float32)
    ea = rng.standard_normal((E, Fe)).astype(np.float32) if Fe else None
    return synth.Batch(gp, x, ei, ea, np.zeros(len(gp) - 1, np.float32))


def _check(m, b):
    ref = oracle.csr_build(b.graph_ptr, b.edge_index, b.num_nodes)
    N, E = b.num_nodes, b.num_edges
    for k, i, n in [("rowptr", 0, N + 1), ("csr_src", 1, E), ("csr_eid", 2, E), ("deg", 3, N),
                    ("srcptr", 4, N + 1), ("t2csr", 5, E), ("node_graph", 6, N)]:
        if n:
            assert np.array_equal(m.fetch(i, 0, (n,)).cpu().numpy(), getattr(ref, k)), k


@pytest.mark.parametrize("N,E,Fe,maxd,per", [
    (1, 0, 1, 4, 30), (1, 3, 0, 4, 30), (63, 100, 2, 4, 30), (256, 512, 1, 4, 30),
    (257, 512, 1, 4, 30), (256, 513, 1, 15, 1), (2048, 4096, 3, 4, 30), (2049, 4096, 1, 20, 2049),
    (1000, 4097, 1, 5, 30), (6144, 12288, 1, 4, 30), (6145, 12288, 1, 4, 30),
    (6144, 12289, 1, 15, 60), (6144, 6000, 4, 4, 1)])
def test_size_classes(N, E, Fe, maxd, per):
    b = _batch(N + E, N, E, Fe, per, min(maxd, 12))
    small = _batch(3, 40, 60, Fe, cap=min(maxd, 12))
    m = _hg().Model(1, 16, 9, Fe, maxd, 0, 0, 1.0)
    for x in (b, small, b): # a context's buffers, reused by other sizes
        m.prepare(_hg().DeviceBatch.from_host(x), validate=True)
        _check(m, x)
    m.close()


# one batch per class of the build; the bad value lies where a workgroup of its
# own copies the input, or where the first one does
@pytest.mark.parametrize("N,E", [(60, 100), (1500, 3000), (6000, 12000), (7000, 14000)])
def test_errors(N, E):
    good = _batch(N, N, E, 1)
    m = _hg().Model(1, 16, 9, 1, 4, 0, 0, 1.0)

    def err(**kw):
        b = synth.Batch(**{**dict(graph_ptr=good.graph_ptr, x=good.x, edge_index=good.edge_index,
                                  edge_attr=good.edge_attr, y=good.y), **kw})
        with pytest.raises(Exception) as e:
            m.prepare(_hg().DeviceBatch.from_host(b), validate=True)
        m.prepare(_hg().DeviceBatch.from_host(good), validate=True)
        return str(e.value)

    x = good.x.copy(); x[N - 1, 8] = np.inf
    assert "non-finite" in err(x=x)
    ea = good.edge_attr.copy(); ea[E // 2, 0] = np.nan
    assert "non-finite" in err(edge_attr=ea)
    for v in (-1, N, 2 ** 31 - 1):
        ei = good.edge_index.copy(); ei[0, E - 1] = v
        assert "out of range" in err(edge_index=ei)
    ei = good.edge_index.copy(); ei[:, 7] = (0, N - 1)
    assert "crosses graphs" in err(edge_index=ei)
    ei = good.edge_index.copy(); ei[:, :6] = 0
    assert "max_degree" in err(edge_index=ei)
    gp = good.graph_ptr.copy(); gp[1] = gp[2]
    assert "graph_ptr" in err(graph_ptr=gp)
    m.close()
