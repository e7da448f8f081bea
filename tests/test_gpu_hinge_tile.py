"""The shared-variable hinge at every lane shape (rows of 8 to 64 lanes per
workgroup, chosen from the number of factors and their dimension), at ragged
factor counts, at the smallest and largest dimensions, with and without
alpha = 1, and with variables in an order that needs the offset list.
Eight iterations from a random (z, u) against the FP64 oracle: z, u, x in
norm and element by element and r, FP64 within 1e-9 and FP32 within 1e-4
(the averages contract: rounding does not grow)."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from paper_1603_02526_amd import admm as A
from tests import parity as P

pytestmark = pytest.mark.gpu

# factors, dimension (FP32; FP64 has half as many factors per workgroup)
SHAPES = [(65_300, 3), (66_000, 31), (32_700, 32), (33_000, 1), (16_400, 63), (8_200, 127), (8_500, 64),
          (1, 1), (31, 15), (33, 255), (257, 200), (700, 128), (2_049, 7)]


def _shuffled(p, seed):
    """The same problem with its variables renumbered at random."""
    perm = np.random.default_rng(seed).permutation(p.n_vars).astype(np.int32)
    for g in p.groups:
        g.var_ids = perm[g.var_ids]
    return p


@pytest.mark.parametrize("prec", [A.FP32, A.FP64])
@pytest.mark.parametrize("n,d", SHAPES)
@pytest.mark.parametrize("alpha,shuffle", [(1.0, False), (1.3, True)])
def test_hinge_lane_shapes(prec, n, d, alpha, shuffle):
    if alpha != 1.0 and n > 40_000:
        pytest.skip("the lane shape is covered with fewer factors")
    p = W.svm(n if prec == A.FP32 else (n + 1) // 2, d, seed=d)
    if shuffle:
        p = _shuffled(p, 3)
    rng = np.random.default_rng(9)
    z0, u0 = 0.3 * rng.standard_normal(p.n_vars), 0.1 * rng.standard_normal(p.n_slots)
    g = A.Graph.from_problem(p, precision=prec, alpha=alpha, driver=A.DRIVER_LAUNCHES)
    o = O.OracleGraph(p, alpha=alpha)
    g.set_state(z0, u0)
    o.set_state(z0, u0)
    g.run(8)
    o.run(8)
    tol = 1e-9 if prec == A.FP64 else 1e-4
    P.check(P.errors(g.z(), g.u(), g.x(), o.z, o.u, o.x, o.slot_z), tol)
    r, ro = g.residuals()[0], o.residuals()[0]
    assert abs(r - ro) <= tol * (ro + float(np.max(np.abs(o.z))))
