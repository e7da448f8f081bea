"""Shared-variable hinge with an infinite dual on one factor's b edge: the
factor's step is one of its bounds (0 or C), so after an iteration w is finite
and matches the FP64 oracle; only b is not.  Sizes whose d + 1 edges do not
fill the lanes of a factor, whose spare lanes read the b edge again."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from paper_1603_02526_amd import admm as A
from tests.helpers import rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [A.FP32, A.FP64])
@pytest.mark.parametrize("driver", [A.DRIVER_AUTO, A.DRIVER_GRAPH])
@pytest.mark.parametrize("n,d,alpha", [(300, 5, 1.0), (300, 5, 1.5), (129, 40, 1.0), (40, 130, 1.0)])
@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_infinite_dual_on_b(prec, driver, n, d, alpha, sign):
    p = W.svm(n, d, seed=3)
    p.alpha = alpha
    off, row = 0, None
    for g in p.groups:
        if g.kind == "hinge":
            row = off
            break
        off += int(np.sum(p.var_dims[g.var_ids]))
    u0 = 0.01 * np.random.default_rng(4).standard_normal(p.n_slots)
    for f in (0, n // 2, n - 1):
        u0[row + f * (d + 1) + d] = sign * np.inf
    z0 = 0.1 * np.random.default_rng(5).standard_normal(len(p.z0))
    g = A.Graph.from_problem(p, precision=prec, driver=driver)
    o = O.OracleGraph(p)
    for s in (g, o):
        s.set_state(z0, u0)
        s.run(1)
    want, got = o.z, g.z()
    assert np.isfinite(want[:d]).all() and not np.isfinite(want[d])
    assert not np.isfinite(got[d])
    assert np.isfinite(got[:d]).all(), got[:d]
    assert rel(got[:d], want[:d]) < (1e-12 if prec == A.FP64 else 1e-5)
