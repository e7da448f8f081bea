"""What the resident driver admits, when it is asked for, does not follow how
a shared hinge is split into workgroups: rows of all factors padded to 64 and
a partial sum per 128 factors up to 32 components, 256 above, against the 96
KB of its limit.  Sizes on both sides of the limit whose split needs more or
less than that."""
import pytest

import workloads as W
from paper_1603_02526_amd import admm as A


def _finalize(p, **kw):
    g = A.Graph.from_problem(p, device=None, **kw)
    try:
        g.finalize(0)
    except A.AdmmError as e:
        if e.status != A.E_NO_DEVICE:
            return e.status, None
    return A.OK, g.info()


@pytest.mark.parametrize("prec,n,d,fits", [
    (A.FP32, 257, 23, True), (A.FP32, 289, 23, True), (A.FP32, 320, 23, True), (A.FP32, 321, 23, False),
    (A.FP32, 1, 128, False), (A.FP32, 20, 150, False), (A.FP32, 32, 213, False),
    (A.FP64, 1, 64, False), (A.FP64, 9, 103, False), (A.FP64, 16, 192, False)])
def test_shared_hinge(prec, n, d, fits):
    status, info = _finalize(W.svm(n, d, seed=1), precision=prec, driver=A.DRIVER_RESIDENT)
    assert status == (A.OK if fits else A.E_UNSUPPORTED)
    if fits:
        assert info["driver"] == A.DRIVER_RESIDENT and info["resident_lds_bytes"] > 0


@pytest.mark.gpu
@pytest.mark.parametrize("prec,n,d", [(A.FP32, 257, 23), (A.FP32, 320, 23), (A.FP64, 100, 23)])
def test_admitted_graph_runs(prec, n, d):
    """Admitted with an image that is up to 1.2 KB over the limit: FP32
    rounding of eight iterations 1e-4, FP64 1e-9, as the resident driver's
    other tests."""
    import numpy as np

    import oracle as O
    from tests.helpers import rel
    p = W.svm(n, d, seed=1)
    g = A.Graph.from_problem(p, precision=prec, driver=A.DRIVER_RESIDENT)
    o = O.OracleGraph(p)
    u0 = 0.02 * np.random.default_rng(1).standard_normal(p.n_slots)
    for s in (g, o):
        s.set_state(p.z0, u0)
        s.run(8)
    tol = 1e-9 if prec == A.FP64 else 1e-4
    assert rel(g.z(), o.z) < tol and rel(g.u(), o.u) < tol
