"""General hinge and margin of more than 32 components in the resident driver,
where a thread takes a factor: components in registers up to 64, two sweeps
over memory above.  Against the FP64 oracle with the resident driver's bounds
(FP64 1e-9; FP32 1e-4 over eight iterations)."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from paper_1603_02526_amd import admm as A
from tests import parity as P

pytestmark = pytest.mark.gpu


def _hinge(n, d):
    """Hinge factors on overlapping windows of scalar variables."""
    p = W.svm(n, d, seed=1)
    g = [g for g in p.groups if g.kind == "hinge"][0]
    nv = 2 * (d + 1)
    g.var_ids = ((np.arange(d + 1)[None, :] + 3 * np.arange(n)[:, None]) % nv).astype(np.int32)
    p.var_dims = np.ones(nv, np.int32)
    p.z0 = np.zeros(nv)
    return p


def _margin(n, d):
    """Margin factors of one vector w, one bias and a slack each."""
    p = W.svm_copies(n, d, seed=2)
    g = [g for g in p.groups if g.kind == "margin"][0]
    ids = np.stack([np.zeros(n), np.ones(n), 2 + np.arange(n)], 1).astype(np.int32)
    groups = [W.FactorGroup("margin", ids, g.params), W.FactorGroup("minerr", ids[:, 2:].copy(), np.array([0.1]), shared=True),
              W.FactorGroup("l2", ids[:1, :1].copy(), np.array([1.0]), shared=True)]
    return W.Problem("margin", np.array([d, 1] + [1] * n, np.int32), groups, np.zeros(d + 1 + n))


@pytest.mark.parametrize("prec,d", [(A.FP32, d) for d in (32, 33, 63, 64, 65, 66)] + [(A.FP64, d) for d in (32, 33, 36)])
@pytest.mark.parametrize("alpha", [1.0, 1.4])
@pytest.mark.parametrize("make", [_hinge, _margin])
def test_wide_factors_match_oracle(make, d, prec, alpha):
    p = make(7, d)
    p.alpha = alpha
    g = A.Graph.from_problem(p, precision=prec, driver=A.DRIVER_RESIDENT)
    o = O.OracleGraph(p)
    u0 = 0.02 * np.random.default_rng(1).standard_normal(p.n_slots)
    z0 = 0.1 * np.random.default_rng(2).standard_normal(len(p.z0))
    for s in (g, o):
        s.set_state(z0, u0)
        s.run(8)
    tol = 1e-9 if prec == A.FP64 else 1e-4
    P.check(P.errors(g.z(), g.u(), g.x(), o.z, o.u, o.x, o.slot_z), tol)
    for a, b in zip(g.residuals(), o.residuals()):
        assert abs(a - b) <= tol * (b + float(np.max(np.abs(o.z))))
