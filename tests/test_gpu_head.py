"""Pooling and the graph head, one operation at a time: one, two and four graphs
a workgroup (batches around 512 and 1024 graphs, last groups partly empty), widths
that divide the workgroup and that do not, inputs off the 16-byte grid."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2207_11333_amd import synth

pytestmark = pytest.mark.gpu


def _rel(a, r):
    return float((a.double().cpu() - r).norm() / r.norm().clamp_min(1e-30))


@pytest.mark.parametrize("B", [1, 3, 511, 512, 513, 1023, 1025, 1030])
@pytest.mark.parametrize("H,off", [(16, 0), (48, 1), (128, 0), (240, 0), (256, 3), (512, 0)])
def test_head(B, H, off):
    from paper_2207_11333_amd import hgnn
    rng = np.random.default_rng(B + H)
    n = rng.integers(1, 9, size=B)
    n[0] = 70
    gp = np.append(0, np.cumsum(n)).astype(np.int32)
    N = int(gp[-1])
    b = synth.Batch(gp, np.zeros((N, 9), np.float32), np.zeros((2, 0), np.int32),
                    np.zeros((0, 1), np.float32), np.zeros(B, np.float32))
    m = hgnn.Model(1, H, 9, 1, 4, 0, 0, 1.0)
    m.prepare(hgnn.DeviceBatch.from_host(b), validate=True)
    hb = torch.tensor(rng.standard_normal(N * H + off), dtype=torch.float32)
    wb = torch.tensor(rng.standard_normal(H * H + 2 * H + 1) / np.sqrt(H), dtype=torch.float32)
    go = torch.tensor(rng.standard_normal(B), dtype=torch.float32)
    h = hb.cuda()[off:].view(N, H).detach().requires_grad_()
    w = wb.cuda().requires_grad_()
    pred = hgnn.PoolHeadFunction.apply(h, w, m)
    dh, dw = torch.autograd.grad(pred, (h, w), go.cuda())

    hd = hb[off:].view(N, H).double().requires_grad_()
    wd = wb.double().requires_grad_()
    seg = torch.repeat_interleave(torch.arange(B), torch.tensor(n))
    g = torch.zeros(B, H, dtype=torch.float64).index_add(0, seg, hd) / torch.tensor(n)[:, None]
    W1, b1 = wd[:H * H].view(H, H), wd[H * H:H * H + H]
    z = g @ W1.T + b1
    ref = torch.relu(z) @ wd[H * H + H:H * H + 2 * H] + wd[-1]
    rdh, rdw = torch.autograd.grad(ref, (hd, wd), go.double())
    print(f"B={B} H={H}: pred {_rel(pred.detach(), ref.detach()):.1e} dh {_rel(dh, rdh):.1e} "
          f"dw {_rel(dw, rdw):.1e} smallest hidden value {float(z.detach().abs().min()):.1e}")
    assert _rel(pred.detach(), ref.detach()) <= 1e-5
    assert _rel(dh, rdh) <= 1e-5
    assert _rel(dw, rdw) <= 1e-5
    m.close()
