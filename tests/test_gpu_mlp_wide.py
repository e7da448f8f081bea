"""Networks and batches large enough for 64-wide tiles (four workgroups per CU
of them; the loss layer by its size) and for fewer splits of the batch, with
sizes that no tile divides, against the FP64 oracle network with the same bf16
operand rounding (the bounds of the other network tests: 1e-3 relative, loss
1e-4); the training step at the edge sizes against Adam applied to the
gradients; and the workspace of a large network."""
import numpy as np
import pytest

from oracle import warmstart as WS
from tests.helpers import rel

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _net(n_in, hid, n_out, batch, seed=5):
    from paper_1603_02526_amd import mlp as MLPm
    net = MLPm.MLP(n_in, hid, n_out, max_batch=batch)
    flat = MLPm.init_params(n_in, hid, n_out, 7, out_scale=1.0)
    net.set_params(flat)
    rng = np.random.default_rng(seed)
    mean, sd = rng.standard_normal(n_out).astype(np.float32), rng.uniform(0.5, 2, n_out).astype(np.float32)
    net.set_output_scaling(mean, sd)
    x = rng.standard_normal((batch, n_in)).astype(np.float32)
    tg = rng.standard_normal((batch, n_out)).astype(np.float32)
    return net, flat, mean, sd, x, tg


# layers 64 wide: hidden x batch or outputs x batch from 1024 tiles of 64 x 64;
# loss 64 wide: (tiles) x hidden from 2^21; splits 8, 4, 2 and 1
@pytest.mark.parametrize("n_in,hid,n_out,batch", [
    (5, 130, 1030, 3900), (7, 1030, 65, 3850), (3, 600, 2050, 8000), (70, 1100, 1400, 300), (5, 2100, 900, 200)])
def test_wide_tiles_match_oracle(n_in, hid, n_out, batch):
    net, flat, mean, sd, x, tg = _net(n_in, hid, n_out, batch)
    xd, td = torch.tensor(x, device="cuda"), torch.tensor(tg, device="cuda")
    y = torch.zeros((batch, n_out), device="cuda")
    g, loss = torch.zeros(net.n_params, device="cuda"), torch.zeros(1, device="cuda")
    net.forward(xd, y)
    net.grads(xd, td, g, loss)
    torch.cuda.synchronize()
    params = WS.unflatten(flat, n_in, hid, n_out)
    m64, s64, x, tg = (a.astype(np.float64) for a in (mean, sd, x, tg))
    yo, _ = WS.mlp_forward(params, x, bf16=True, mean=m64, sd=s64)
    assert rel(y.cpu().numpy(), yo) < 1e-3
    lo, go = WS.mlp_loss_grad(params, x, tg, bf16=True, mean=m64, sd=s64)
    assert abs(loss.item() - lo) < 1e-4 * abs(lo)
    for a, b in zip(WS.unflatten(g.cpu().numpy(), n_in, hid, n_out), go):
        assert rel(a, b) < 1e-3


@pytest.mark.parametrize("n_in,hid,n_out,batch", [(1, 1, 1, 1), (5, 65, 129, 65), (129, 96, 300, 32), (8, 64, 65, 1025),
                                                  (5, 2100, 900, 200)])
def test_training_step_is_adam_on_the_gradients(n_in, hid, n_out, batch):
    """Two steps with the decay rates and bias corrections in FP32, as the
    step has them; m, v and the step in FP32: the update within 1e-5 of lr."""
    net, flat, _, _, x, tg = _net(n_in, hid, n_out, batch)
    xd, td = torch.tensor(x, device="cuda"), torch.tensor(tg, device="cuda")
    g = torch.zeros(net.n_params, device="cuda")
    lr, p = 1e-2, flat.astype(np.float64)
    m = v = np.zeros_like(p)
    for k in (1, 2):
        net.grads(xd, td, g, None)
        gk = g.cpu().numpy().astype(np.float64)
        net.train_step(xd, td, lr)
        b1, b2, one = np.float32(0.9), np.float32(0.999), np.float32(1)
        c1, c2 = (float(one - np.float32(b ** k)) for b in (0.9, 0.999))
        m = float(b1) * m + float(one - b1) * gk
        v = float(b2) * v + float(one - b2) * gk * gk
        step = lr * (m / c1) / (np.sqrt(v / c2) + 1e-8)
        got = net.get_params().astype(np.float64)
        # lr (1e-5 of the step's size, 4e-4 where the square of a tiny gradient is denormal in FP32) and p's rounding
        tol = lr * np.where(np.abs(gk) > 1e-15, 1e-5, 1.1) + 1.2e-7 * np.abs(p)
        assert np.max(np.abs(got - (p - step)) / tol) <= 1
        p = got


def test_large_network_workspace():
    """A network whose tiles fill the chip keeps one copy of its gradients:
    parameters, two moments and the copy, and the activations."""
    from paper_1603_02526_amd import mlp as MLPm
    torch.zeros(1, device="cuda")
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    net = MLPm.MLP(1024, 4096, 1024, max_batch=512)
    used = before - torch.cuda.mem_get_info()[0]
    assert used < 4 * (4 * net.n_params + 512 * (4 * 4096 + 2 * 1024)) + (64 << 20)
