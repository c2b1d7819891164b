"""The captured iteration of step-level fp64 solves, which holds the caller's
arrays: taken and replayed for the arrays of the solve before, and for no others."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2111_11788_amd as mm
from workloads import Workload


# 32^3: above the whole solves in one workgroup, which capture nothing.  Eager,
# captured and replayed, replayed; then another kappa (eager), another solution
# array, and that one again (captured anew), with work of the caller's in between
@pytest.mark.parametrize("solver,deg,direction", [(0, 1, True), (0, 2, True), (0, 2, False), (1, 1, True)])
def test_solves_replay_on_the_same_arrays_only(solver, deg, direction):
    n, B = 32, 3
    wl = Workload("graph", n0=n, levels=1, sigma2=1.0, corr_len=0.3, n_modes=20, qoi=0, rtol=1e-9, max_iter=3000,
                  solver=solver, precision=0, batch=B)

    def context():
        c = mm.Context(wl, cheb_degree=deg, arena_bytes=256 << 20)
        if not direction:
            c.set_tuning(fuse=c.tuning()["fuse"] & ~mm.FUSE_DIRECTION)
        return c

    ctx = context()
    kaps = {"A": ctx.field(n, ctx.draw_xi(0, 0, B)), "B": ctx.field(n, ctx.draw_xi(0, 50, B))}
    want = {}
    for k, kap in kaps.items():
        one = context()
        want[k] = one.solve(n, kap)
        one.close()
    us = [torch.zeros((B, mm.grid_stride(n)), dtype=torch.float64, device="cuda") for _ in range(2)]
    for k, j in (("A", 0), ("A", 0), ("A", 0), ("B", 0), ("A", 1), ("A", 1), ("A", 1), ("B", 1)):
        us[0].mul_(0.5)   # the caller's own work between solves
        us[1].mul_(0.5)
        it = np.zeros(B, dtype=np.int32)
        rc = mm.lib().mlmc_solve(ctx.h, n, B, kaps[k].data_ptr(), us[j].data_ptr(), it.ctypes.data)
        assert rc == 0
        assert torch.equal(us[j], want[k][0]) and np.array_equal(it, want[k][1]), (k, j)
    # new values in the same arrays: the replayed iteration reads what is there
    kaps["A"].copy_(kaps["B"])
    for _ in range(2):
        rc = mm.lib().mlmc_solve(ctx.h, n, B, kaps["A"].data_ptr(), us[0].data_ptr(), it.ctypes.data)
        assert rc == 0 and torch.equal(us[0], want["B"][0])
    ctx.close()
