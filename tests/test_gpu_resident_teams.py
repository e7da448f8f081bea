"""The resident driver's team kernel (several blocks of a pass side by side)
at block counts around the number of teams and with every factor kind it
takes: the same blocks and arithmetic as separate launches of the same plan
on one workgroup, so against the FP64 oracle it keeps the resident driver's
bounds (FP64 1e-9; FP32 1e-4 over eight iterations), with residuals, general
alpha, group weights, a split run and a state import."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from paper_1603_02526_amd import admm as A
from tests import parity as P

pytestmark = pytest.mark.gpu


def _spread(n, shape, seed):
    """Disks on a coarse lattice with contacts: a well-conditioned packing."""
    p = W.packing(n, shape, 0.05, seed=seed)
    rng = np.random.default_rng(seed)
    k = int(np.ceil(np.sqrt(n)))
    g = np.stack(np.meshgrid(np.arange(k), np.arange(k)), -1).reshape(-1, 2)[:n]
    p.z0[0::3], p.z0[1::3] = ((g + 0.5) / k + 0.05 / k * rng.uniform(-1, 1, (n, 2))).T
    p.z0[2::3] = rng.uniform(0.4, 0.55, n) / k
    return p


def _equal_chain(n, seed):
    """n vectors of two components tied by equality, with L2, box, minimal-
    error and quadratic terms: every separable kind and the equality pairs."""
    rng = np.random.default_rng(seed)
    i = np.arange(n, dtype=np.int32)
    groups = [W.FactorGroup("equal", np.stack([i[:-1], i[1:]], 1), np.zeros((0,)), shared=True),
              W.FactorGroup("l2", i[:, None], np.array([0.3]), shared=True),
              W.FactorGroup("box", i[:, None], np.array([-0.5, 0.7]), shared=True),
              W.FactorGroup("minerr", i[::2, None].copy(), np.array([0.01]), shared=True),
              W.FactorGroup("quad", i[:, None], rng.uniform(0.1, 1, (n, 2)))]
    return W.Problem("chain", np.full(n, 2, np.int32), groups, rng.standard_normal(2 * n))


def _case(name):
    if name.startswith("chain"):
        return _equal_chain(int(name[5:]), 3)
    return _spread(int(name[4:]), "square", 5)


@pytest.mark.parametrize("prec", [A.FP32, A.FP64])
@pytest.mark.parametrize("name", ["pack2", "pack10", "pack23", "pack26", "chain2", "chain150", "chain300"])
@pytest.mark.parametrize("alpha,weights", [(1.0, False), (1.4, True)])
def test_team_kernel_matches_oracle(prec, name, alpha, weights):
    p = _case(name)
    p.alpha = alpha
    if weights:
        for k, g in enumerate(p.groups):
            g.rho = 1.0 + 0.5 * k
    g = A.Graph.from_problem(p, precision=prec)
    if g.info()["driver"] != A.DRIVER_RESIDENT:
        pytest.skip("graph too large for the resident driver")
    o = O.OracleGraph(p)
    u0 = 0.02 * np.random.default_rng(1).standard_normal(p.n_slots)
    g.set_state(p.z0, u0)
    o.set_state(p.z0, u0)
    g.run(5)
    g.run(3)
    o.run(8)
    tol = 1e-9 if prec == A.FP64 else 1e-4
    P.check(P.errors(g.z(), g.u(), g.x(), o.z, o.u, o.x, o.slot_z), tol)
    for a, b in zip(g.residuals(), o.residuals()):
        assert abs(a - b) <= tol * (b + float(np.max(np.abs(o.z))))
