"""A NaN in an initial state stays a NaN on its way through the horizon, one
time step further with each iteration: no clamp makes it an infinity, no later
step is touched, and the other instances of the batch keep their results."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("iters", [1, 2, 3, 7])
@pytest.mark.parametrize("T", [9, 30, 40, 150])
@pytest.mark.parametrize("n,m,box", [(3, 1, 1.0), (6, 3, 0.0), (12, 4, 0.5)])
def test_nan_state(n, m, box, T, iters):
    from paper_1603_02526_amd import mpc as M
    rng = np.random.default_rng(7)
    A, B = W.mpc_system(rng, n, m)
    insts = [W.MPCInstance(T, n, m, A, B, rng.standard_normal(n), np.ones(n), np.full(m, 0.1), box) for _ in range(3)]

    def solve():
        b = M.MPCBatch(insts)
        x0 = torch.tensor(b.pack_x0([i.x0 for i in insts]), device="cuda")
        z = torch.zeros(b.z_total, dtype=torch.float32, device="cuda")
        it = torch.zeros(b.n_inst, dtype=torch.int32, device="cuda")
        b.solve_state(x0, z, it, tol=1e-30, max_iter=iters)
        assert np.all(it.cpu().numpy() == -iters)
        return [zi.reshape(T, n + m) for zi in b.split_z(z.cpu().numpy())]

    want = solve()
    insts[1].x0 = insts[1].x0.copy()
    insts[1].x0[0] = np.nan
    got = solve()
    reach = min(T, iters)
    assert np.isnan(got[1][:reach]).all(), got[1][:reach]
    assert np.isfinite(got[1][reach:]).all()
    for k in (0, 2):
        assert np.array_equal(got[k], want[k])
