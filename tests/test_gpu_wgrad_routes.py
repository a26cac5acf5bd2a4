"""The routes of the weight gradients against one another: every layer's in one
launch, a layer's two products on the second stream (FP32 k_wgrad, BF16
k_gemm_tn_tr) and both in one launch.  All sum the same chunks in the same order,
so the gradients are equal bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2207_11333_amd import synth

pytestmark = pytest.mark.gpu


def _hg():
    from paper_2207_11333_amd import hgnn
    return hgnn


def _grads(b, params, L, H, prec, recompute=0, maxd=4, kind="pna", fail=0):
    hg = _hg()
    m = hg.Model(L, H, 9, 1, maxd, prec, recompute, 1.08, kind=kind)
    m.set_params(params)
    m.debug_fail_alloc(fail)  # 1: without the buffers of the one launch
    db = hg.DeviceBatch.from_host(b)
    pred, loss = torch.empty(b.num_graphs, device="cuda"), torch.empty(1, device="cuda")
    m.forward(db, pred, loss, validate=True)
    m.backward()
    g = m.grads().cpu().numpy()
    m.close()
    return g


# hidden widths from 29 chunks a product down to 2 (dealt to the XCDs by whole
# chunks and, the few FP32 ones of the wide layers, by rows of tiles), batches on
# both sides of the limit of two products in one launch, and from a few nodes (one
# row chunk) up; degrees up to 12 (13 buckets)
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("H,graphs,lo,hi,maxd", [
    (64, 2, 5, 9, 4), (128, 200, 30, 40, 4), (176, 100, 30, 40, 4), (192, 40, 30, 40, 12),
    (240, 100, 30, 40, 4), (256, 30, 30, 40, 4), (256, 140, 30, 40, 4), (320, 60, 30, 40, 4),
    (384, 50, 30, 40, 4), (512, 1, 40, 40, 4), (512, 20, 30, 40, 4), (512, 60, 30, 40, 4)])
def test_routes_agree(prec, H, graphs, lo, hi, maxd):
    b = synth.make_batch(11, graphs, lo, hi, 1)
    p = synth.init_params(synth.ModelShape(2, H, 9, 1), 12)
    one = _grads(b, p, 2, H, prec, maxd=maxd)
    assert np.isfinite(one).all() and np.abs(one).max() > 0
    assert np.array_equal(one, _grads(b, p, 2, H, prec, maxd=maxd, fail=1))
    assert np.array_equal(one, _grads(b, p, 2, H, prec, recompute=1, maxd=maxd))


@pytest.mark.parametrize("kind", ["sage", "cgcnn"])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("H,graphs", [(256, 40), (384, 20), (512, 3), (512, 60)])
def test_other_layer_kinds(kind, prec, H, graphs):
    b = synth.make_batch(13, graphs, 30, 40, 1)
    p = synth.init_gc_params(kind, 2, H, 14, edge_feat=1)
    one = _grads(b, p, 2, H, prec, kind=kind)
    assert np.isfinite(one).all() and np.abs(one).max() > 0
    assert np.array_equal(one, _grads(b, p, 2, H, prec, kind=kind, fail=1))


# FP32 products of H = 512 come in two chunks of half the nodes each: above 8192
# nodes the layers go one at a time
@pytest.mark.parametrize("graphs,launches", [(225, 1), (245, 2)])
def test_long_chunks_go_layer_by_layer(graphs, launches):
    hg = _hg()
    b = synth.make_batch(15, graphs, 33, 37, 1)
    assert (b.num_nodes < 8192) == (launches == 1)
    p = synth.init_params(synth.ModelShape(1, 512, 9, 1), 16)
    m = hg.Model(1, 512, 9, 1, 4, 0, 0, 1.08)
    m.set_params(p)
    db = hg.DeviceBatch.from_host(b)
    pred, loss = torch.empty(b.num_graphs, device="cuda"), torch.empty(1, device="cuda")
    n = 0
    for site in ("update_wgrad", "message_wgrad"):
        m.timer_start(site, 8)
        m.forward(db, pred, loss)
        m.backward()
        n += m.timer_read()[1]
    assert n == launches
    got = m.grads().cpu().numpy()
    m.close()
    if launches == 1:  # else a failed allocation of the workspace is an error
        assert np.array_equal(got, _grads(b, p, 1, 512, 0, fail=1))
    assert np.array_equal(got, _grads(b, p, 1, 512, 0, recompute=1))


def _against_the_oracle(b, H, Fe, maxd):
    import oracle
    from test_gpu_parity import (ELEM_FP32, TAU_FP32, gpu_decisions, grad_report, make_model, maxrel,
                                 rel, run_train_step)
    L, delta = 2, 1.3
    shape = synth.ModelShape(L, H, 9, Fe)
    params = synth.init_params(shape, 18 + Fe)
    m = make_model(L, H, Fe, 0, 0, delta, maxd)
    out = run_train_step(m, b, params)
    rec = oracle.forward(params, b, L, H, delta)
    g_ref, _, _ = oracle.backward(rec, hint=gpu_decisions(m, L, H, b.num_nodes, b.num_graphs),
                                  tau=TAU_FP32)
    g = out["grads"].cpu().numpy()
    assert rel(out["pred"].cpu().numpy(), rec.y) <= 1e-5
    rep, erep = grad_report(m, g, g_ref, shape), grad_report(m, g, g_ref, shape, elementwise=True)
    print(f"H={H} Fe={Fe}: worst gradient {max(rep.values()):.2e}, element-wise {max(erep.values()):.2e}")
    assert max(rep.values()) <= 1e-5
    assert max(erep.values()) <= ELEM_FP32
    m.close()


# A batch too large for the one launch: the fused backward leaves each layer's
# second-stream products to be joined two layers on, the per-operation entries join
# every layer at once.  Several steps back to back, so that a step's products still run
# while the next one's chain begins.  (The loss gradient is formed by torch on one side
# and by the head kernel on the other, as in test_deferred_joins_match_per_layer_joins,
# whose batch is below the limit, and with that test's tolerances.)
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("H", [64, 80])
def test_deferred_joins_of_a_large_batch(prec, H):
    hg = _hg()
    from test_gpu_parity import rel
    b = synth.make_batch(19, 500, 30, 50, 1)
    assert b.num_nodes >= 16384 and b.num_nodes * H > 640 * 1024
    L = 5
    p = synth.init_params(synth.ModelShape(L, H, 9, 1), 20)
    m = hg.Model(L, H, 9, 1, 4, prec, 0, 1.08)
    m.set_params(p)
    db = hg.DeviceBatch.from_host(b)
    pred, loss = torch.empty(b.num_graphs, device="cuda"), torch.empty(1, device="cuda")
    for _ in range(3):
        m.forward(db, pred, loss)
        m.backward()
    fused = m.grads()
    net = hg.PNANet(m, p)
    for _ in range(3):
        net.zero_grad()
        out = net(db)
        ((out - db.y) ** 2).mean().backward()
    torch.cuda.synchronize()
    assert torch.equal(out.detach(), pred)
    r = rel(net.packed_grad().cpu().numpy(), fused.cpu().numpy())
    print(f"H={H} prec={prec}: gradient rel {r:.2e}")
    assert r <= (1e-5 if prec else 1e-6)
    m.close()


# Batches of 20,480 nodes or more: the products by themselves on the second stream,
# the De rows left to their column sums.  H = 64 runs k_wgrad, widths that are no
# multiple of 32, and 32, k_gemm_tn (bucketed and plain chunks; 72 and 24 of them whole to an
# XCD), except H = 208 with 16 chunks; no other route takes such a batch, so against the
# FP64 oracle (decision replay, the FP32 path's tolerances).
@pytest.mark.parametrize("H,Fe,maxd", [(64, 1, 4), (32, 1, 4), (48, 1, 4), (80, 2, 4), (48, 0, 4), (48, 1, 20),
                                       (48, 1, 7), (208, 1, 7), (208, 1, 15)])
def test_large_fp32_against_the_oracle(H, Fe, maxd):
    b = synth.make_batch(17 + Fe, 620, 20, 50, Fe)
    assert b.num_nodes >= 20480
    _against_the_oracle(b, H, Fe, maxd)


# Without buckets the widths between 288 and 384 run k_gemm_tn at every size: one
# node, one row chunk, several
@pytest.mark.parametrize("H,graphs,lo,hi", [(304, 1, 1, 1), (336, 2, 5, 9), (368, 60, 20, 40)])
def test_middle_widths_without_buckets(H, graphs, lo, hi):
    _against_the_oracle(synth.make_batch(21, graphs, lo, hi, 1), H, 1, 20)
