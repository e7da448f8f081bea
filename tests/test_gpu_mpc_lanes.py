"""Batches that keep the device busy with equal work run with one lane per time
step; the arithmetic is that of the tiles, so instances of every state size
and horizon among thousands of small ones keep the bits (z, duals, iterations)
that they have in a batch of their own."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _batch(insts):
    from paper_1603_02526_amd import mpc as M
    b = M.MPCBatch(insts)
    return b, torch.tensor(b.pack_x0([i.x0 for i in insts]), device="cuda")


def _solves(b, x0, noise):
    """Cold from nothing, from a state, and from a prediction."""
    z, u = (torch.zeros(n, dtype=torch.float32, device="cuda") for n in (b.z_total, b.u_total))
    out = []
    it = torch.zeros(b.n_inst, dtype=torch.int32, device="cuda")
    b.solve_state(x0, z, it, u_out=u, tol=1e-4, max_iter=90)
    out.append((z.cpu().numpy(), u.cpu().numpy(), it.cpu().numpy()))
    z2, u2 = torch.zeros_like(z), torch.zeros_like(u)
    b.solve_state(x0, z2, it, z_init=z, u_init=u, u_out=u2, tol=1e-5, max_iter=40)
    out.append((z2.cpu().numpy(), u2.cpu().numpy(), it.cpu().numpy()))
    b.solve(x0, z2, it, z_init=z + noise, dual=True, tol=1e-4, max_iter=60)
    out.append((z2.cpu().numpy(), u2.cpu().numpy(), it.cpu().numpy()))
    return out


def _instances(shapes, seed):
    rng = np.random.default_rng(seed)
    out = []
    for T, n, m, box in shapes:
        A, B = W.mpc_system(rng, n, m)
        out.append(W.MPCInstance(T, n, m, A, B, rng.standard_normal(n), np.ones(n), np.full(m, 0.1), box))
    return out


LONG = [(T, n, m, box) for n, m, box in ((1, 1, 1.0), (4, 2, 0.0), (5, 1, 1.0), (6, 4, 0.5), (7, 2, 0.0), (8, 3, 1.0),
                                         (9, 3, 1.0), (10, 2, 0.5), (11, 4, 1.0), (12, 4, 0.0))
        for T in (1, 63, 64, 65, 128, 129, 192, 256)]
SHORT = [(T, n, m, box) for n, m, box in ((1, 1, 1.0), (4, 4, 0.0), (5, 2, 0.5)) for T in (1, 2, 63, 64, 65, 127, 128)]


@pytest.mark.parametrize("shapes,count,resident", [(LONG, 24576, 512), (SHORT, 24576, 1024)])
def test_same_bits_as_alone(shapes, count, resident):
    insts = _instances(shapes, 91)
    filler = _instances([(50, 4, 2, 1.0)] * 4, 92)
    rng = np.random.default_rng(93)
    more = [W.MPCInstance(50, 4, 2, f.A, f.B, rng.standard_normal(4), f.q, f.r, f.u_box)
            for f in (filler[k % 4] for k in range(count))]
    few, x_few = _batch(insts)
    many, x_many = _batch(insts + more)
    # the larger batch runs on lanes (two waves per SIMD: two workgroups of four per CU, four of two)
    assert many.plan()["resident"] == resident and few.plan()["resident"] != resident
    noise = 4e-3 * torch.randn(many.z_total, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    a = _solves(few, x_few, noise[:few.z_total])
    b = _solves(many, x_many, noise)
    for (z, u, it), (z2, u2, it2) in zip(a, b):
        assert np.array_equal(it, it2[:len(it)])
        assert np.array_equal(z, z2[:len(z)])
        assert np.array_equal(u, u2[:len(u)])


def test_nan_state_on_lanes():
    """A NaN initial state stays in its instance, one step further with each
    iteration, as on tiles."""
    insts = _instances([(T, n, 2, 1.0) for T in (9, 64, 100) for n in (3, 8)], 94)
    filler = _instances([(50, 4, 2, 1.0)], 95)[0]
    for i in insts:
        i.x0 = i.x0.copy()
        i.x0[0] = np.nan
    b, x0 = _batch(insts + [filler] * 24576 + _instances([(130, 4, 1, 1.0)], 96))
    assert b.plan()["resident"] == 512
    z = torch.zeros(b.z_total, dtype=torch.float32, device="cuda")
    it = torch.zeros(b.n_inst, dtype=torch.int32, device="cuda")
    b.solve(x0, z, it, tol=1e-30, max_iter=3)
    parts = b.split_z(z.cpu().numpy())
    for i, zi in zip(insts, parts):
        zi = zi.reshape(i.T, i.n + i.m)
        assert np.isnan(zi[:3]).all() and np.isfinite(zi[3:]).all(), (i.T, i.n)
    assert np.isfinite(np.concatenate(parts[len(insts):])).all()
    assert np.all(it.cpu().numpy() == -3)
