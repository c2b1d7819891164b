"""How a launch's planes are split over workgroups depends on the batch; a
sample's bits do not."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2111_11788_amd as mm
from workloads import Workload


def _wl(**kw):
    base = dict(name="split", n0=8, levels=1, sigma2=1.0, corr_len=0.3, n_modes=20, qoi=0, rtol=1e-9, max_iter=3000,
                solver=0, precision=0, batch=16)
    base.update(kw)
    return Workload(**base)


def _same_bits_alone(ctx, n, kap, of):
    u, it = ctx.solve(n, kap)
    for a, b in of:
        v, iv = ctx.solve(n, kap[a:b].contiguous())
        assert torch.equal(v, u[a:b]) and np.array_equal(iv, it[a:b])


# 128^3: 8 planes a workgroup for one sample, 16 to 64 for a batch; 256^3: 16
# against 32; degree 1 takes the fused residual update, 2 the separate one, Jacobi
# the plain loop
@pytest.mark.parametrize("n,B,prec,solver,deg", [(128, 40, 0, 0, 1), (128, 40, 0, 0, 2), (128, 70, 1, 0, 1),
                                                 (128, 70, 1, 0, 2), (128, 20, 0, 1, 1), (256, 4, 1, 0, 2),
                                                 (256, 4, 0, 0, 1)])
def test_large_meshes_sum_in_an_order_of_their_own(n, B, prec, solver, deg):
    wl = _wl(n0=n, precision=prec, solver=solver, rtol=1e-9 if solver == 0 else 1e-5)
    ctx = mm.Context(wl, cheb_degree=deg, arena_bytes=24 << 30)
    kap = ctx.field(n, ctx.draw_xi(0, 0, B))
    _same_bits_alone(ctx, n, kap, [(0, 1), (B - 1, B), (1, 4)])
    ctx.close()


# meshes whose default is a whole solve in one workgroup, on the level-by-level
# kernels: split stencil launches and sums per unit of planes
@pytest.mark.parametrize("n,B,prec,deg", [(4, 300, 1, 1), (8, 70, 0, 1), (8, 1500, 1, 2), (16, 700, 1, 1),
                                          (16, 700, 1, 2), (16, 1300, 0, 1)])
def test_small_meshes_on_the_level_kernels(n, B, prec, deg):
    ctx = mm.Context(_wl(n0=n, precision=prec), cheb_degree=deg, arena_bytes=2 << 30)
    ctx.set_tuning(fuse=ctx.tuning()["fuse"] & ~mm.FUSE_SOLVE, vsmall_fp32=0, vsmall_fp64=0)
    kap = ctx.field(n, ctx.draw_xi(0, 0, B))
    _same_bits_alone(ctx, n, kap, [(0, 1), (B - 1, B), (1, 4)])
    ctx.close()
