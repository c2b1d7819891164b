"""Step-level calls of several contexts on the null stream: in the order of the
calls, as the caller's memory is."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2111_11788_amd as mm
from workloads import Workload


@pytest.mark.parametrize("n,count", [(32, 400), (64, 60)])
def test_two_contexts_queue_their_fields_in_order(n, count):
    # `a` queues fields whose outputs are freed at once; the field of `b` takes the
    # memory of the last of them and must not be written over by it
    wl = Workload("streams", n0=n, levels=1, sigma2=1.0, corr_len=0.3, n_modes=64, qoi=0, rtol=1e-8, max_iter=100,
                  solver=0, precision=1, batch=8)
    a, b = mm.Context(wl, arena_bytes=64 << 20), mm.Context(wl, arena_bytes=64 << 20)
    xa, xb = a.draw_xi(0, 0, count), b.draw_xi(0, 10000, count)
    want, want32 = b.field(n, xb, want32=True)
    torch.cuda.synchronize()
    for _ in range(3):
        for _ in range(30):
            a.field(n, xa, want32=True)
        k, k32 = b.field(n, xb, want32=True)
        torch.cuda.synchronize()
        assert torch.equal(k, want) and torch.equal(k32, want32)
        del k, k32
    a.close()
    b.close()


def test_queued_calls_and_solves_of_one_context_are_ordered():
    # field and V-cycle (null stream), solve (the context's stream), and back,
    # without waiting in between, against the same steps with a wait after each
    n, count = 32, 50
    wl = Workload("streams", n0=n, levels=1, sigma2=1.0, corr_len=0.3, n_modes=64, qoi=0, rtol=1e-8, max_iter=100,
                  solver=0, precision=1, batch=count)
    ctx = mm.Context(wl, arena_bytes=1 << 30)

    def steps(wait):
        out = []
        for first in (0, 100, 200):
            xi = ctx.draw_xi(0, first, count)
            wait()
            kap, k32 = ctx.field(n, xi, want32=True)
            wait()
            u, _ = ctx.solve(n, kap)
            y = ctx.apply(n, kap, u)
            wait()
            z = ctx.vcycle_f32(n, k32, y.float())
            wait()
            q = ctx.qoi(n, u)
            wait()
            out += [u, y, z, q]
        torch.cuda.synchronize()
        return out

    want = steps(torch.cuda.synchronize)
    for _ in range(3):
        for g, w in zip(steps(lambda: None), want):
            assert torch.equal(g, w)
    ctx.close()


def test_closing_a_context_waits_for_its_queued_calls():
    n, count = 32, 400
    wl = Workload("streams", n0=n, levels=1, sigma2=1.0, corr_len=0.3, n_modes=64, qoi=0, rtol=1e-8, max_iter=100,
                  solver=0, precision=1, batch=8)
    ctx = mm.Context(wl, arena_bytes=64 << 20)
    xi = ctx.draw_xi(0, 0, count)
    want = ctx.field(n, xi)
    torch.cuda.synchronize()
    k = [ctx.field(n, xi) for _ in range(30)]
    ctx.close()
    assert torch.cuda.current_stream().query()   # nothing left running
    assert all(torch.equal(v, want) for v in (k[0], k[-1]))


def test_kernel_times_of_queued_calls():
    n, count = 32, 400
    wl = Workload("streams", n0=n, levels=1, sigma2=1.0, corr_len=0.3, n_modes=64, qoi=0, rtol=1e-8, max_iter=100,
                  solver=0, precision=1, batch=8)
    ctx = mm.Context(wl, arena_bytes=64 << 20)
    xi = ctx.draw_xi(0, 0, count)
    ctx.set_profiling(True)
    k = [ctx.field(n, xi) for _ in range(20)]
    launches, ms, nbytes = ctx.kernel_time("FIELD")[:3]
    assert launches == 20 and ms > 0.0
    ctx.close()
    del k
