"""What serving reports for requests that do not converge: pools that solve a
request whole in one workgroup (up to 16^3, the default) against the same pools
stepping one iteration at a time."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2111_11788_amd as mm
from workloads import Workload


def _serve(wl, reqs, whole, slots):
    ctx = mm.Context(wl, arena_bytes=1 << 30)
    if not whole:
        ctx.set_tuning(fuse=ctx.tuning()["fuse"] & ~mm.FUSE_SOLVE)
    ctx.serve_start(slots)
    out = []
    for _ in range(2):   # the second time on slots that gave up the first
        tickets = [ctx.submit(l, s) for l, s in reqs]
        res = ctx.wait(tickets)
        out.append([res[t] for t in tickets])
    ctx.serve_stop()
    ctx.close()
    for a, b in zip(*out):
        assert a["status"] == b["status"] and a["iters"] == b["iters"]
    return out[0]


def _wl(**kw):
    base = dict(name="status", n0=16, levels=2, sigma2=1.0, corr_len=0.3, n_modes=32, qoi=0, rtol=1e-9, max_iter=400,
                solver=0, precision=1, batch=8)
    base.update(kw)
    return Workload(**base)


# a slot is given up after 4 max_iter + 1 iterations: 5 to 13 here, where 16^3
# solves need 9 to 14 of them
@pytest.mark.parametrize("max_iter", [1, 2, 3])
def test_the_iteration_limit_is_the_stepping_pools(max_iter):
    wl = _wl(max_iter=max_iter)
    reqs = [(0, s) for s in range(24)]
    a, b = _serve(wl, reqs, True, [8, 0]), _serve(wl, reqs, False, [8, 0])
    for x, y in zip(a, b):
        assert x["status"] == y["status"] and x["status"] in (0, -4)
        assert x["iters"] == y["iters"] <= 4 * max_iter + 1
        if x["status"] == 0:
            assert x["q_fine"] == y["q_fine"]
    assert max_iter > 1 or all(r["status"] == -4 for r in a)


# a tolerance below what fp64 can reach: every iteration of the limit is spent,
# also where that takes more refinements than a batch call makes (30)
def test_a_tolerance_out_of_reach_spends_the_limit():
    wl = _wl(rtol=1e-30, max_iter=30)
    for whole in (True, False):
        for r in _serve(wl, [(0, s) for s in range(4)], whole, [4, 0]):
            assert r["status"] == -4 and r["iters"] == 121 and np.isfinite(r["q_fine"])


# kappa that overflows makes the residual NaN: its own request ends with
# MLMC_E_NONFINITE, in the whole-solve pool and in the stepping one of 32^3
@pytest.mark.parametrize("whole", [True, False])
@pytest.mark.parametrize("level", [0, 1])
def test_overflow_is_reported(level, whole):
    wl = _wl(sigma2=1e7)
    for r in _serve(wl, [(level, s) for s in range(6)], whole, [4, 4]):
        assert r["status"] == -5
