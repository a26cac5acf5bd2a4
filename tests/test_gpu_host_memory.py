"""Host memory allocated right after a context, a server or a graph store was closed
keeps its contents: nothing of what these freed is written to later."""
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2207_11333_amd import graphstore, hgnn, synth

pytestmark = pytest.mark.gpu


def _train(db, kind):
    m = hgnn.Model(2, 80 if kind == "sage" else 64, 9, 1, 4, 0, 0, 1.08, kind=kind)
    m.set_params((torch.rand(m.num_params) - .5) * .1)
    pred = torch.empty(db.num_graphs, device="cuda")
    for _ in range(2):
        m.forward(db, pred, torch.empty(1, device="cuda"))
        m.backward()
    torch.cuda.synchronize()
    m.close()


def _serve(b):
    m = hgnn.Model(2, 32, 9, 1, 4, 0, 0, 1.08)
    m.serve_start(hbm_budget_bytes=1 << 30, num_lanes=4)
    t, out, end = m.serve_submit(b), None, time.time() + 30
    while out is None and time.time() < end:
        out = m.serve_poll(t, b.num_graphs)
    assert np.isfinite(out).all()
    m.close()


def _store(path):
    s = hgnn.GraphStore(str(path))
    for _ in range(3):
        s.next()
    torch.cuda.synchronize()
    s.close()


def test_untouched_after_close(tmp_path):
    b = synth.make_batch(7, 40, 5, 30, 1)
    db = hgnn.DeviceBatch.from_host(synth.make_batch(8, 1100, 5, 30, 1))
    graphstore.write_store(str(tmp_path / "s.bin"), [b, b])
    for _ in range(12):
        for close in (lambda: _train(db, "sage"), lambda: _train(db, "pna"),
                      lambda: _serve(b), lambda: _store(tmp_path / "s.bin")):
            close()
            # sizes around those that the closed objects leave on the heap
            arrays = [np.full(n, 384, np.int64) for n in range(64, 264) for _ in range(8)]
            time.sleep(0.005)
            assert all((a == 384).all() for a in arrays)
