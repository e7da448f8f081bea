"""Solves of one batch that overlap on two streams share its work queue and
may spoil each other's results (the header asks for them to be ordered); a
solve that starts after them has to handle every instance again, whatever the
overlapping launches' sizes were, with a queue and with a workgroup per item.
Its result: that of a batch of its own (the same arithmetic: equal bits)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _arrays(b):
    return (torch.full((b.z_total,), 7.0, dtype=torch.float32, device="cuda"),
            torch.full((b.n_inst,), 7, dtype=torch.int32, device="cuda"))


@pytest.mark.parametrize("mode", ["cold", "state", "dual"])
@pytest.mark.parametrize("grids", [(1, 4), (4, 1), (2, 3), (3, 5), (2, 6), (6, 4)])
def test_solve_after_overlapping_solves(grids, mode):
    from paper_1603_02526_amd import mpc as M
    insts = W.mpc_batch(6, seed=81, T_range=(40, 48))
    b, own = M.MPCBatch(insts), M.MPCBatch(insts)
    x0 = torch.tensor(b.pack_x0([i.x0 for i in insts]), device="cuda")
    zi, ii = _arrays(own)
    own.solve(x0, zi, ii, tol=1e-2, max_iter=50)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    scratch = [_arrays(b) for _ in streams]
    torch.cuda.synchronize()
    for g, s, (z, it) in zip(grids, streams, scratch):
        b.set_plan(4, 0, g)
        b.solve(x0, z, it, tol=1e-30, max_iter=3000, stream=s.cuda_stream)
    torch.cuda.synchronize()

    def solve(batch):
        z, it = _arrays(batch)
        if mode == "cold":
            batch.solve(x0, z, it, tol=1e-4, max_iter=300)
        elif mode == "state":
            batch.solve_state(x0, z, it, z_init=zi, tol=1e-4, max_iter=300)
        else:
            batch.solve(x0, z, it, z_init=zi, dual=True, tol=1e-4, max_iter=300)
        return z.cpu().numpy(), it.cpu().numpy()

    want = solve(own)
    for g in (1, 4, 6, 4):
        b.set_plan(4, 0, g)
        got = solve(b)
        assert np.array_equal(got[1], want[1]), (g, got[1], want[1])
        assert np.array_equal(got[0], want[0]), g
