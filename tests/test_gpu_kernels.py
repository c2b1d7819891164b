"""Edges of the kernels' tiles and of the rules that choose them, against the
oracle or against the general form of the same kernel."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2111_11788_amd as mm
from oracle import field, rng
from workloads import Workload


def _wl(**kw):
    base = dict(name="k", n0=8, levels=1, sigma2=1.0, corr_len=0.3, n_modes=20, qoi=0, rtol=1e-12, max_iter=3000,
                solver=0, precision=0, batch=16)
    base.update(kw)
    return Workload(**base)


# meshes below 64^3: 4 samples to a workgroup at 4^3 and 8^3, one at 16^3, a
# quarter of one at 32^3; counts on both sides of that, K1 <= 8, 16 and 32, and
# mode counts at which the workgroup's coefficients no longer fit (the row-wise form)
@pytest.mark.parametrize("n,M,corr,count", [(4, 8, 0.5, 1), (4, 20, 0.2, 5), (4, 512, 0.1, 4), (8, 3, 0.5, 4),
                                            (8, 128, 0.2, 9), (8, 1, 0.3, 1), (8, 300, 0.2, 13), (16, 20, 0.1, 1),
                                            (16, 512, 0.2, 3), (16, 1500, 0.2, 2), (32, 64, 0.5, 1), (32, 512, 0.1, 3),
                                            (32, 700, 0.2, 2), (8, 2000, 0.1, 5)])
def test_field_below_64_matches_oracle(n, M, corr, count):
    # tolerance: the sums differ in order only; exp turns an absolute error of
    # a few 1e-15 times |g| <= ~10 into a relative one
    wl = _wl(n0=n, n_modes=M, corr_len=corr)
    ctx = mm.Context(wl, arena_bytes=64 << 20)
    xi = ctx.draw_xi(0, 7, count)
    k, k32 = ctx.field(n, xi, want32=True)
    want = field.kappa(n, corr, 1.0, M, rng.draw_xi(wl.seed, 0, 7, count, M))
    got = k.cpu().numpy()
    assert np.max(np.abs(got - want) / want) < 1e-13
    assert np.array_equal(k32.cpu().numpy(), got.astype(np.float32))
    # a sample's field does not depend on its batch
    assert torch.equal(ctx.field(n, xi[count - 1:])[0], k[count - 1])
    ctx.close()


@pytest.mark.parametrize("n,deg", [(4, 2), (8, 3), (16, 2), (32, 2), (32, 4), (64, 2), (128, 2)])
@pytest.mark.parametrize("prec", [0, 1])
def test_zero_step_inside_the_second_step_gives_the_stored_bits(n, deg, prec):
    # Chebyshev degree >= 2: the zero-start smoothing step formed inside the
    # second one, against the step stored by its own kernel
    ctx = mm.Context(_wl(n0=n), cheb_degree=deg, arena_bytes=1 << 30)
    dt = torch.float64 if prec == 0 else torch.float32
    g = torch.Generator(device="cuda").manual_seed(n + deg)
    kap = torch.exp(torch.randn((2, n ** 3), generator=g, dtype=torch.float64, device="cuda")).to(dt)
    r = mm.to_grid(torch.randn((2, (n - 1) ** 3), generator=g, dtype=torch.float64, device="cuda").to(dt), n)
    f = ctx.vcycle if prec == 0 else ctx.vcycle_f32
    out = []
    for fuse in (mm.FUSE_PROLONG | mm.FUSE_RESTRICT | mm.FUSE_PRESMOOTH, mm.FUSE_PROLONG | mm.FUSE_RESTRICT):
        ctx.set_tuning(fuse=fuse, vsmall_fp32=0, vsmall_fp64=0)
        out.append(f(n, kap, r))
    assert bool(torch.isfinite(out[0]).all()) and torch.equal(out[0], out[1])
    ctx.close()


@pytest.mark.parametrize("solver", [0, 1])
def test_fp64_solves_on_other_arrays(solver):
    # one context, one batch size, different kappa and solution arrays: the
    # captured iteration is taken again for them
    n = 8
    ctx = mm.Context(_wl(n0=n, solver=solver, rtol=1e-9), arena_bytes=64 << 20)
    kap = ctx.field(n, ctx.draw_xi(0, 0, 6))
    keep = [ctx.solve(n, kap[k:k + 1].contiguous()) for k in (0, 3, 5, 0)]
    for k, (u, it) in zip((0, 3, 5, 0), keep):
        one = mm.Context(_wl(n0=n, solver=solver, rtol=1e-9), arena_bytes=64 << 20)
        w, iw = one.solve(n, kap[k:k + 1].contiguous())
        assert torch.equal(u, w) and it[0] == iw[0]
        one.close()
    ctx.close()


# the planes of a small launch are split over workgroups (32^3: chunks of 4
# planes for one sample, one chunk for 1100), a sample's sums are not: the same
# sample alone and in a batch that fills the chip has the same bits
@pytest.mark.parametrize("n,B,prec,deg", [(8, 70, 0, 1), (16, 700, 0, 2), (16, 700, 1, 1), (32, 1100, 1, 2),
                                          (32, 600, 0, 1), (64, 300, 1, 1), (64, 130, 0, 2)])
def test_split_planes_leave_a_samples_bits(n, B, prec, deg):
    ctx = mm.Context(_wl(n0=n, precision=prec, rtol=1e-9), cheb_degree=deg, arena_bytes=12 << 30)
    xi = ctx.draw_xi(0, 0, B)
    kap = ctx.field(n, xi)
    u, it = ctx.solve(n, kap)
    for k in (0, B - 1):
        u1, it1 = ctx.solve(n, kap[k:k + 1].contiguous())
        assert torch.equal(u1[0], u[k]) and it1[0] == it[k]
    u3, it3 = ctx.solve(n, kap[1:4].contiguous())
    assert torch.equal(u3, u[1:4]) and np.array_equal(it3, it[1:4])
    ctx.close()


# whole solves in one workgroup against the level-by-level kernels, both to a
# true relative residual of 1e-12: the iterates differ by at most the condition
# number of the Jacobi-scaled operator (~ n^2 times the contrast of kappa,
# below 1e4) times twice that
@pytest.mark.parametrize("n", [4, 8, 16])
@pytest.mark.parametrize("prec,solver,deg", [(0, 0, 1), (0, 0, 3), (0, 1, 1), (1, 0, 1), (1, 0, 2), (1, 0, 3)])
def test_whole_solves_match_the_level_kernels(n, prec, solver, deg):
    ctx = mm.Context(_wl(n0=n, precision=prec, solver=solver), cheb_degree=deg, arena_bytes=256 << 20)
    kap = ctx.field(n, ctx.draw_xi(0, 3, 5))
    fuse = ctx.tuning()["fuse"]
    got = {}
    for f in (fuse | mm.FUSE_SOLVE, fuse & ~mm.FUSE_SOLVE):
        ctx.set_tuning(fuse=f)
        got[f] = ctx.solve(n, kap)
    (u, it), (w, iw) = got.values()
    assert float((u - w).norm() / w.norm()) <= 2e-8
    assert np.abs(it - iw).max() <= 1
    # a sample alone, and boundary positions
    ctx.set_tuning(fuse=fuse | mm.FUSE_SOLVE)
    assert torch.equal(ctx.solve(n, kap[2:3].contiguous())[0][0], u[2])
    assert float(u.abs().sum()) == pytest.approx(float(mm.from_grid(u, n).abs().sum()), rel=1e-15)
    ctx.close()


@pytest.mark.parametrize("n", [4, 8, 16])
@pytest.mark.parametrize("prec,solver", [(0, 0), (0, 1), (1, 0)])
def test_whole_solves_report_their_status(n, prec, solver):
    # a NaN coefficient ends its own sample only; a cap of 2 iterations is reported
    wl = _wl(n0=n, precision=prec, solver=solver)
    ctx = mm.Context(wl, arena_bytes=256 << 20)
    kap = ctx.field(n, ctx.draw_xi(0, 3, 4))
    good, _ = ctx.solve(n, kap)
    kap[1, 5] = float("nan")
    u = torch.zeros_like(good)
    it = np.zeros(4, dtype=np.int32)
    rc = mm.lib().mlmc_solve(ctx.h, n, 4, kap.data_ptr(), u.data_ptr(), it.ctypes.data)
    assert rc == -5   # MLMC_E_NONFINITE
    assert torch.equal(u[[0, 2, 3]], good[[0, 2, 3]])
    ctx.close()
    short = mm.Context(wl, arena_bytes=256 << 20, max_iter=2)
    xi = short.draw_xi(0, 3, 4)
    _, it = short.solve(n, short.field(n, xi), allow_noconv=True)
    assert it.max() <= 2
    with pytest.raises(mm.MLMCError) as e:
        short.solve(n, short.field(n, xi))
    assert e.value.code == -4
    short.close()


# the coarse end of the V-cycle (and with it the 16^3 preconditioner) keeps the
# level-by-level result: fp32 rounding of a few steps apart
@pytest.mark.parametrize("n,deg", [(4, 1), (8, 2), (16, 1), (16, 2), (16, 4), (32, 2)])
@pytest.mark.parametrize("prec", [0, 1])
def test_single_kernel_vcycle_matches_the_level_kernels(n, deg, prec):
    ctx = mm.Context(_wl(n0=n), cheb_degree=deg, arena_bytes=256 << 20)
    dt = torch.float64 if prec == 0 else torch.float32
    g = torch.Generator(device="cuda").manual_seed(n + deg)
    kap = torch.exp(torch.randn((3, n ** 3), generator=g, dtype=torch.float64, device="cuda")).to(dt)
    r = mm.to_grid(torch.randn((3, (n - 1) ** 3), generator=g, dtype=torch.float64, device="cuda").to(dt), n)
    f = ctx.vcycle if prec == 0 else ctx.vcycle_f32
    z = f(n, kap, r)
    ctx.set_tuning(vsmall_fp32=0, vsmall_fp64=0)
    w = f(n, kap, r)
    assert float((z - w).norm() / w.norm()) <= (1e-13 if prec == 0 else 2e-5)
    ctx.close()


# more than 128 samples take the form of the single-kernel V-cycle that two
# workgroups per CU fit: the same operations in the same order
@pytest.mark.parametrize("n,deg", [(16, 1), (16, 3), (32, 2)])
@pytest.mark.parametrize("B", [129, 300])
def test_single_kernel_vcycle_of_a_large_batch_keeps_a_samples_bits(n, deg, B):
    ctx = mm.Context(_wl(n0=n, precision=1), cheb_degree=deg, arena_bytes=2 << 30)
    g = torch.Generator(device="cuda").manual_seed(n + deg)
    kap = torch.exp(torch.randn((B, n ** 3), generator=g, dtype=torch.float64, device="cuda")).float()
    r = mm.to_grid(torch.randn((B, (n - 1) ** 3), generator=g, dtype=torch.float64, device="cuda").float(), n)
    z = ctx.vcycle_f32(n, kap, r)
    for a in range(0, B, 100):
        assert torch.equal(ctx.vcycle_f32(n, kap[a:a + 100].contiguous(), r[a:a + 100].contiguous()), z[a:a + 100])
    ctx.close()


# the fp64 refinement of a 256^3 solve (rows of two waves in LDS, with and
# without the update the fp32 solve owes): the residual it stops on is the true
# one, b = h^3 at every interior node, up to the rounding of two fp64 evaluations
@pytest.mark.parametrize("B,deg,direction", [(1, 1, True), (2, 2, True), (3, 1, False)])
def test_refinement_at_256_stops_on_the_true_residual(B, deg, direction):
    n, rtol = 256, 1e-9
    ctx = mm.Context(_wl(n0=n, precision=1, rtol=rtol), cheb_degree=deg, arena_bytes=16 << 30)
    if not direction:
        ctx.set_tuning(fuse=ctx.tuning()["fuse"] & ~mm.FUSE_DIRECTION)
    kap = ctx.field(n, ctx.draw_xi(0, 0, B))
    u, _ = ctx.solve(n, kap)
    b = mm.to_grid(torch.full((B, (n - 1) ** 3), n ** -3.0, dtype=torch.float64, device="cuda"), n)
    r = b - ctx.apply(n, kap, u)
    for s in range(B):
        assert float(r[s].norm() / b[s].norm()) <= rtol * 1.01
    ctx.close()


# the streaming kernels run several loads ahead: spans below, at and above that
@pytest.mark.parametrize("n", [2, 4, 16, 32, 64, 128])
def test_domain_average_of_every_span(n):
    ctx = mm.Context(_wl(n0=n), arena_bytes=1 << 30)
    g = torch.Generator(device="cuda").manual_seed(n)
    v = torch.rand((3, (n - 1) ** 3), generator=g, dtype=torch.float64, device="cuda")
    q = np.asarray(ctx.qoi(n, mm.to_grid(v, n)).cpu())
    assert np.allclose(q, v.sum(1).cpu().numpy() / n ** 3, rtol=1e-12, atol=0)
    ctx.close()


# a V-cycle has no sums: however its levels' planes are split (down to 8 of them
# a workgroup at 128^3, 4 at 64^3 and 2 below for one sample), the bits are the same
@pytest.mark.parametrize("n,B,deg", [(32, 600, 2), (64, 200, 1), (128, 12, 1), (128, 12, 3)])
@pytest.mark.parametrize("prec", [0, 1])
def test_vcycle_of_one_sample_has_the_bits_of_a_batch(n, B, deg, prec):
    ctx = mm.Context(_wl(n0=n, precision=prec), cheb_degree=deg, arena_bytes=12 << 30)
    dt = torch.float64 if prec == 0 else torch.float32
    g = torch.Generator(device="cuda").manual_seed(n + deg)
    kap = torch.exp(torch.randn((B, n ** 3), generator=g, dtype=torch.float64, device="cuda")).to(dt)
    r = mm.to_grid(torch.randn((B, (n - 1) ** 3), generator=g, dtype=torch.float64, device="cuda").to(dt), n)
    f = ctx.vcycle if prec == 0 else ctx.vcycle_f32
    z = f(n, kap, r)
    for s in (0, B - 1):
        assert torch.equal(f(n, kap[s:s + 1].contiguous(), r[s:s + 1].contiguous())[0], z[s])
    ctx.close()


# results above the pinned staging of a round (and of a solve) are copied
# straight to the caller's memory: the same numbers
@pytest.mark.parametrize("level,count", [(0, 20000), (1, 18000)])
def test_results_beyond_the_staging_are_the_staged_ones(level, count):
    ctx = mm.Context(_wl(n0=4, levels=2, precision=1, rtol=1e-8), arena_bytes=6 << 30)
    whole = ctx.sample_level(level, 0, count)
    half = count // 2
    parts = [ctx.sample_level(level, 0, half), ctx.sample_level(level, half, count - half)]
    for w, a, b in zip(whole, *parts):
        assert np.array_equal(np.asarray(w), np.concatenate([a, b]))
    kap = ctx.field(4, ctx.draw_xi(0, 0, 20000))
    it = ctx.solve(4, kap)[1]
    assert np.array_equal(it[:9000], ctx.solve(4, kap[:9000].contiguous())[1])
    ctx.close()
