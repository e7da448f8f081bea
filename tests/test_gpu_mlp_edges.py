"""The network's products at the edges of their tiles (64 rows, 32 or 64
columns, chunks of 128 of the summed index, the batch shared by up to eight
workgroups), with rows that are not 16-byte aligned and inputs that start in
the middle of a buffer, against the FP64 oracle network with the same bf16
operand rounding: forward and gradients within 1e-3 relative, the loss
within 1e-4 (the bounds of the other network tests; both sides round the same
operands, a different order of fp32 sums may flip single bf16 roundings)."""
import numpy as np
import pytest

from oracle import warmstart as WS
from tests.helpers import rel

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n_in,hid,n_out,batch,offset", [
    (1, 1, 1, 1, 0), (3, 31, 33, 63, 1), (4, 32, 32, 64, 0), (5, 65, 129, 65, 3), (33, 130, 64, 257, 2),
    (128, 128, 127, 129, 0), (129, 96, 300, 32, 4), (8, 256, 1100, 511, 0), (8, 64, 65, 1025, 1)])
def test_edges_match_oracle(n_in, hid, n_out, batch, offset):
    from paper_1603_02526_amd import mlp as MLPm
    net = MLPm.MLP(n_in, hid, n_out, max_batch=batch + 3)
    flat = MLPm.init_params(n_in, hid, n_out, 7, out_scale=1.0)
    net.set_params(flat)
    rng = np.random.default_rng(5)
    mean, sd = rng.standard_normal(n_out).astype(np.float32), rng.uniform(0.5, 2, n_out).astype(np.float32)
    net.set_output_scaling(mean, sd)
    x = rng.standard_normal((batch + offset, n_in)).astype(np.float32)
    tg = rng.standard_normal((batch + offset, n_out)).astype(np.float32)
    xd, td = torch.tensor(x, device="cuda")[offset:], torch.tensor(tg, device="cuda")[offset:]
    x, tg = x[offset:].astype(np.float64), tg[offset:].astype(np.float64)
    y = torch.zeros((batch, n_out), device="cuda")
    g, loss = torch.zeros(net.n_params, device="cuda"), torch.zeros(1, device="cuda")
    net.forward(xd, y)
    net.grads(xd, td, g, loss)
    torch.cuda.synchronize()
    params = WS.unflatten(flat, n_in, hid, n_out)
    m64, s64 = mean.astype(np.float64), sd.astype(np.float64)
    yo, _ = WS.mlp_forward(params, x, bf16=True, mean=m64, sd=s64)
    assert rel(y.cpu().numpy(), yo) < 1e-3
    lo, go = WS.mlp_loss_grad(params, x, tg, bf16=True, mean=m64, sd=s64)
    assert abs(loss.item() - lo) < 1e-4 * abs(lo)
    for a, b in zip(WS.unflatten(g.cpu().numpy(), n_in, hid, n_out), go):
        assert rel(a, b) < 1e-3 if np.linalg.norm(b) > 0 else np.all(a == 0)
    # again, and as a training step from the same parameters: the same bits
    g2 = torch.zeros_like(g)
    net.grads(xd, td, g2, None)
    torch.cuda.synchronize()
    assert torch.equal(g, g2)
