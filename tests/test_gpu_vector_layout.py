"""Margin, equality and separable factors on vector variables, where one
offset per factor edge stands for the components' offsets, and the same
factors where it cannot: variables of several dimensions, or lists of
different lengths (a fifth contribution moves a variable's list to another
region).  Dimensions around the register bounds (32, 64) and a workgroup
(256), and factor counts whose slots end inside a workgroup.  Eight
iterations from a random (z, u) against the FP64 oracle: z, u, x in norm and
element by element and r, FP64 within 1e-9 and FP32 within 1e-4 (as for the
other averages contracts: rounding does not grow)."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from paper_1603_02526_amd import admm as A
from tests import parity as P

pytestmark = pytest.mark.gpu


def _copies(n, d, form):
    """n points with their own copy of w in a chain and a box per copy;
    "lists": four more boxes on every third copy; "dims": one more variable
    of another dimension, with a box and in an equality of its own."""
    p = W.svm_copies(n, d, seed=d)
    i = np.arange(n, dtype=np.int32)
    ids, lo = i, -0.1 - 0.01 * (i % 7)
    if form == "lists":
        ids, lo = np.repeat(i[::3], 4), np.full(4 * len(i[::3]), -0.05)
    p.groups.append(W.FactorGroup("box", ids[:, None], np.stack([lo, lo + 0.3], 1)))
    if form == "dims":
        v = p.n_vars
        p.var_dims = np.concatenate([p.var_dims, np.full(2, d + 1, np.int32)])
        p.z0 = np.zeros(int(p.var_dims.sum()))
        for g in p.groups:
            extra = {"box": [v], "equal": [v, v + 1], "l2": [v]}.get(g.kind)
            if extra:
                g.var_ids = np.concatenate([g.var_ids, np.array([extra], np.int32)])
                if g.kind == "box":
                    g.params = np.concatenate([g.params, [[-1.0, 1.0]]])
    return p


@pytest.mark.parametrize("prec", [A.FP32, A.FP64])
@pytest.mark.parametrize("form", ["vector", "lists", "dims"])
@pytest.mark.parametrize("n,d,alpha", [(1, 2, 1.0), (300, 1, 1.0), (129, 2, 1.3), (700, 31, 1.0), (64, 32, 1.3),
                                       (515, 33, 1.0), (90, 65, 1.0), (70, 200, 1.3),
                                       # margins large enough to be split over lanes
                                       (33_000, 2, 1.3), (16_400, 7, 1.0), (4_001, 31, 1.0), (3_900, 32, 1.3),
                                       (3_745, 33, 1.0), (2_000, 65, 1.3), (1_000, 129, 1.0), (511, 255, 1.0)])
def test_vector_offsets(prec, form, n, d, alpha):
    p = _copies(n, d, form)
    rng = np.random.default_rng(9)
    z0, u0 = 0.3 * rng.standard_normal(len(p.z0)), 0.1 * rng.standard_normal(p.n_slots)
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


@pytest.mark.parametrize("n,d", [(3, 257), (2, 70_000)])
def test_vector_offsets_long(n, d):
    """Equality and separable factors alone, longer than a workgroup and longer
    than one offset serves, in a chain."""
    i = np.arange(n, dtype=np.int32)
    lo = -0.2 - 0.1 * i
    p = W.Problem(name="chain", var_dims=np.full(n, d, np.int32), z0=np.zeros(n * d), groups=[
        W.FactorGroup("box", i[:, None], np.stack([lo, lo + 0.3], 1)),
        W.FactorGroup("equal", np.stack([i[:-1], i[1:]], 1), np.zeros((0,)), shared=True)])
    rng = np.random.default_rng(9)
    z0, u0 = 0.3 * rng.standard_normal(n * d), 0.1 * rng.standard_normal(p.n_slots)
    g = A.Graph.from_problem(p, precision=A.FP64, driver=A.DRIVER_LAUNCHES)
    o = O.OracleGraph(p)
    g.set_state(z0, u0)
    o.set_state(z0, u0)
    g.run(8)
    o.run(8)
    P.check(P.errors(g.z(), g.u(), g.x(), o.z, o.u, o.x, o.slot_z), 1e-9)


@pytest.mark.parametrize("prec", [A.FP32, A.FP64])
@pytest.mark.parametrize("n,d,alpha", [(1, 1, 1.0), (7, 8, 1.3), (16_400, 32, 1.0), (16_300, 9, 1.3), (300, 33, 1.0),
                                       (65, 64, 1.3), (2_050, 65, 1.0), (130, 128, 1.0), (33, 129, 1.3), (17, 255, 1.0)])
def test_hinge_on_own_variables(prec, n, d, alpha):
    """Hinge factors on differing variables, at every split of a workgroup
    between factors (8 to 64) and their components."""
    p = W.svm(n, d, seed=d)
    rng = np.random.default_rng(9)
    g = next(g for g in p.groups if g.kind == "hinge")
    nv = d + 1 + min(n, 200)
    p.var_dims, p.z0 = np.ones(nv, np.int32), np.zeros(nv)
    g.var_ids = ((np.arange(d + 1)[None, :] * 3 + rng.integers(0, nv, n)[:, None]) % nv).astype(np.int32)
    if nv % 3 == 0:
        g.var_ids = ((np.arange(d + 1)[None, :] + rng.integers(0, nv, n)[:, None]) % nv).astype(np.int32)
    z0, u0 = 0.3 * rng.standard_normal(nv), 0.1 * rng.standard_normal(p.n_slots)
    gr = A.Graph.from_problem(p, precision=prec, alpha=alpha, driver=A.DRIVER_LAUNCHES)
    o = O.OracleGraph(p, alpha=alpha)
    gr.set_state(z0, u0)
    o.set_state(z0, u0)
    gr.run(8)
    o.run(8)
    tol = 1e-9 if prec == A.FP64 else 1e-4
    P.check(P.errors(gr.z(), gr.u(), gr.x(), o.z, o.u, o.x, o.slot_z), tol)
    r, ro = gr.residuals()[0], o.residuals()[0]
    assert abs(r - ro) <= tol * (ro + float(np.max(np.abs(o.z))))
