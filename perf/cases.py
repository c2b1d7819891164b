"""What a user of this library has it do, as cases to be timed.

Each case is one call (or one burst of calls) through the public entry points
of ``paper_2111_11788_amd``, at sizes of the workloads in ``workloads.py`` or
between them: a single sample, the levels of a multilevel run from 8^3 to
256^3, the batched 64^3 workload, and the step-level calls a program that
builds its own solver makes (field, V-cycle, solve), in fp64, in mixed
precision and with the bf16 KLE of the serving workload.

``exact`` evaluates the same quantities in fp64 with NumPy and torch alone
(its own KLE, Philox draw, Q1 operator, Jacobi-PCG and V-cycle).  Iteration
counts of ``sample_level`` are diagnostics of the solver and are not part of
the result; the QoIs and Y are.
"""
import math

import numpy as np
import torch

import paper_2111_11788_amd as mm
import workloads

# the tuning a program that runs the batched 64^3 workload pins (an autotuner pick)
BATCH64_TUNING = {"zvar_fp32": 2, "zvar_fp64": 2, "vsmall_fp32": 16, "vsmall_fp64": 8, "cheb_degree": 1,
                  "max_batch": 256, "graph_batch": 1, "fuse": 447, "lanes": 4}

# fields of a case that are not given take these values
DEFAULTS = {"kind": "sample", "n0": 8, "levels": 1, "level": 0, "count": 1, "M": 128, "corr": 0.2, "sigma2": 1.0,
            "precision": 1, "solver": 0, "degree": 0, "qoi": 0, "forcing": 0, "rtol": 1e-8, "max_batch": 1024,
            "arena_mb": 1024, "pinned": False}


def listed():
    return [
        # the smallest call: one sample of a fine/coarse pair, latency only
        {"name": "one-sample-16", "n0": 8, "levels": 2, "level": 1, "count": 1},
        # a plain MLMC run in fp64 with Jacobi-PCG (4^3, 8^3, 16^3; 200, 50 and 12 samples)
        {"name": "plain-mlmc-fp64", "kind": "estimate", "n0": 4, "levels": 3, "M": 8, "corr": 0.5, "precision": 0,
         "solver": 1, "rtol": 1e-10, "max_batch": 64, "n_fixed": "200,50,12"},
        # the coarsest level of a multilevel run, where the allocation puts most samples
        {"name": "coarse-8", "n0": 8, "levels": 5, "level": 0, "count": 13001, "arena_mb": 8192},
        # a top-up of its next level (16^3 / 8^3 pairs)
        {"name": "topup-16", "n0": 8, "levels": 5, "level": 1, "count": 1131, "arena_mb": 8192},
        # a pilot of 32 samples on a middle level (32^3 / 16^3 pairs)
        {"name": "pilot-32", "n0": 8, "levels": 5, "level": 2, "count": 32, "arena_mb": 8192},
        # the batched 64^3 workload with its pinned tuning
        {"name": "batch-64", "n0": 64, "count": 1024, "M": 64, "corr": 0.3, "qoi": 1, "arena_mb": 20480,
         "pinned": True},
        # the same problem in fp64 at the library's default tuning
        {"name": "batch-64-fp64", "n0": 64, "count": 96, "M": 64, "corr": 0.3, "qoi": 1, "precision": 0,
         "max_batch": 96, "arena_mb": 6144},
        # the largest mesh: a batch of four 256^3 samples
        {"name": "stress-256", "n0": 256, "count": 4, "M": 512, "corr": 0.1, "sigma2": 2.0, "max_batch": 4,
         "arena_mb": 12288},
        # a solve on given coefficients, a few samples of a large mesh
        {"name": "solve-128", "kind": "solve", "n0": 128, "count": 3, "max_batch": 3, "arena_mb": 2048},
        # the preconditioner alone, fp32
        {"name": "vcycle-64", "kind": "vcycle", "n0": 64, "count": 50, "M": 64, "corr": 0.3, "max_batch": 50,
         "arena_mb": 4096},
        # the coefficient field alone, fp64 and its fp32 copy
        {"name": "field-32", "kind": "field", "n0": 32, "count": 777, "M": 256, "arena_mb": 64},
        # a burst of serving requests over 16^3 to 64^3, bf16 KLE
        {"name": "serve-mix", "kind": "serve", "n0": 16, "levels": 3, "count": 400, "M": 256, "precision": 2,
         "max_batch": 64, "arena_mb": 8192, "slots": "1024,256,32"},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["sample", "sample", "sample", "solve", "vcycle", "field", "serve"])
    c = {"kind": kind, "corr": rng.choice([0.1, 0.2, 0.3, 0.5]), "M": rng.choice([8, 20, 64, 100, 128, 256])}
    if kind == "serve":
        c.update(n0=16, levels=3, count=_log_int(rng, 20, 600), M=256, precision=rng.choice([1, 2]), max_batch=64,
                 arena_mb=8192, slots="1024,256,32")
        return c
    if kind == "field":
        n = rng.choice([8, 16, 32, 64, 128])
        c.update(n0=n, count=_log_int(rng, 1, min(4000, (1 << 25) // n ** 3)), precision=rng.choice([0, 1, 1, 2]),
                 arena_mb=64)
        return c
    n = rng.choice([8, 16, 32, 64, 128])
    count = _log_int(rng, 1, max(2, min(6000, (1 << 24) // n ** 3)))
    c.update(n0=n, count=count, degree=rng.choice([0, 0, 1]), precision=rng.choice([0, 1, 1]), max_batch=count,
             arena_mb=8192)
    if kind == "sample":
        c.update(qoi=rng.choice([0, 1]), forcing=rng.choice([0, 0, 0, 1]), max_batch=max(8, count))
        if n >= 16 and rng.random() < 0.6:   # a fine/coarse pair
            c.update(n0=n // 2, levels=2, level=1)
        if n <= 16 and c["precision"] == 0:
            c["solver"] = rng.choice([0, 1])
    return c


def _full(case):
    c = dict(DEFAULTS)
    c.update(case)
    return c


def _first(seed):
    """The first sample index a call takes: each seed its own range."""
    return 1000003 * (seed % 100000)


def _workload(c, seed):
    return workloads.Workload("case", n0=c["n0"], levels=c["levels"], sigma2=c["sigma2"], corr_len=c["corr"],
                              n_modes=c["M"], seed=workloads.DEFAULT_SEED + seed, qoi=c["qoi"], rtol=c["rtol"],
                              solver=c["solver"], precision=c["precision"], forcing=c["forcing"])


def _serve_levels(c, seed):
    """Levels of a burst, weighted 16^-level (the serving mix's law), at least one request of each."""
    rng = np.random.default_rng(seed)
    w = np.array([16.0 ** -l for l in range(c["levels"])])
    lv = rng.choice(c["levels"], size=c["count"], p=w / w.sum())
    lv[:c["levels"]] = np.arange(c["levels"])
    return lv.astype(np.int32)


def _xi(c, seed):
    g = torch.Generator().manual_seed(seed)
    return torch.randn((c["count"], c["M"]), generator=g, dtype=torch.float64)


def _rhs(c, seed, dtype):
    g = torch.Generator(device="cuda").manual_seed(seed + 1)
    return torch.randn((c["count"], (c["n0"] - 1) ** 3), generator=g, dtype=torch.float64, device="cuda").to(dtype)


def prepare(case, seed):
    c = _full(case)
    ctx = mm.Context(_workload(c, seed), arena_bytes=c["arena_mb"] << 20, max_batch=c["max_batch"],
                     cheb_degree=c["degree"])
    if c["pinned"]:
        ctx.set_tuning(**BATCH64_TUNING)
    s = {"case": c, "ctx": ctx, "first": _first(seed)}
    if c["kind"] == "estimate":
        s["n_fixed"] = [int(x) for x in c["n_fixed"].split(",")]
    elif c["kind"] == "serve":
        s["levels"] = _serve_levels(c, seed)
        s["ids"] = np.arange(c["count"], dtype=np.uint64) + np.uint64(s["first"])
        ctx.serve_start([int(x) for x in c["slots"].split(",")])
    elif c["kind"] != "sample":
        s["xi"] = _xi(c, seed).cuda()
        if c["kind"] in ("solve", "vcycle"):
            k, k32 = ctx.field(c["n0"], s["xi"], want32=True)
            s["kappa"] = k if c["kind"] == "solve" or c["precision"] == 0 else k32
        if c["kind"] == "vcycle":
            dt = torch.float64 if c["precision"] == 0 else torch.float32
            s["r"] = mm.to_grid(_rhs(c, seed, dt), c["n0"])
    return s


def run(s):
    c, ctx = s["case"], s["ctx"]
    kind = c["kind"]
    if kind == "sample":
        y, qf, qc, _ = ctx.sample_level(c["level"], s["first"], c["count"])
        return {"y": y, "q_fine": qf, "q_coarse": qc}
    if kind == "estimate":
        ctx.reset_stats()
        nl, est = ctx.estimate(1.0, n_fixed=s["n_fixed"])
        return {"qtilde": est["qtilde"], "var": est["var_qtilde"], "n": nl.astype(np.int64),
                "mean": np.array([l["mean"] for l in est["levels"]]),
                "m2": np.array([l["m2"] for l in est["levels"]])}
    if kind == "solve":
        u, it = ctx.solve(c["n0"], s["kappa"])
        return {"u": u, "iters": it}
    if kind == "vcycle":
        f = ctx.vcycle if c["precision"] == 0 else ctx.vcycle_f32
        return {"z": f(c["n0"], s["kappa"], s["r"])}
    if kind == "field":
        k, k32 = ctx.field(c["n0"], s["xi"], want32=True)
        return {"kappa": k, "kappa32": k32}
    tickets = ctx.submit_batch(s["levels"], s["ids"])
    left, got = len(tickets), []
    while left:
        r = ctx.drain_array(max_results=4096, timeout=1.0)
        left -= len(r)
        got.append(r)
    r = np.concatenate(got)
    r = r[np.argsort(r["ticket"])]
    return {"y": r["y"].copy(), "q_fine": r["q_fine"].copy(), "q_coarse": r["q_coarse"].copy()}


def work(case):
    """Bytes read and written once (draws and coefficients in, results out) and the operations of the
    method's steps: about 50 per node for an operator row or a smoothing step, the V-cycles of ~9 PCG
    iterations (~40 Jacobi iterations) per solve."""
    c = _full(case)
    B, M, n = c["count"], c["M"], c["n0"] << c["level"]

    def cycle(n, deg):
        return sum((m - 1) ** 3 for m in (n >> q for q in range(12)) if m >= 2) * 50.0 * (2 * deg + 1)

    def solve(n):
        if c["solver"] == 1:
            return 40 * 60.0 * (n - 1) ** 3
        return 9 * (cycle(n, c["degree"] or 2) + 60.0 * (n - 1) ** 3)

    def field(n):
        return n ** 3 * 60.0

    def pair(level):
        n = c["n0"] << level
        return solve(n) + field(n) + (solve(n // 2) + field(n // 2) if level else 0.0)

    if c["kind"] == "sample":
        return {"bytes": 24.0 * B, "flops": B * pair(c["level"])}
    if c["kind"] == "estimate":
        ns = [int(x) for x in c["n_fixed"].split(",")]
        return {"bytes": 8.0 * sum(ns), "flops": sum(k * pair(l) for l, k in enumerate(ns))}
    if c["kind"] == "serve":
        lv = _serve_levels(c, 0)
        return {"bytes": 24.0 * B, "flops": sum(pair(int(l)) for l in lv)}
    if c["kind"] == "solve":
        return {"bytes": 8.0 * B * (n ** 3 + (n - 1) ** 3), "flops": B * solve(n)}
    if c["kind"] == "vcycle":
        sz = 8.0 if c["precision"] == 0 else 4.0
        return {"bytes": sz * B * (n ** 3 + 2 * (n - 1) ** 3), "flops": B * cycle(n, c["degree"] or 2)}
    return {"bytes": B * (8.0 * M + 12.0 * n ** 3), "flops": B * field(n)}


# ---------------------------------------------------------------- exact values (fp64, NumPy and torch alone)

def _modes(corr, sigma2, M):
    """The M largest separable modes of the exponential covariance: triples, sqrt(lambda), 1D omega."""
    c = 1.0 / corr
    kmax = 8
    while True:
        om = []
        for q in range(kmax + 1):
            f = (lambda w: c * math.cos(w / 2) - w * math.sin(w / 2)) if q % 2 == 0 else \
                (lambda w: w * math.cos(w / 2) + c * math.sin(w / 2))
            lo, hi = q * math.pi, (q + 1) * math.pi
            s = f(lo + 1e-9) > 0
            for _ in range(200):
                mid = 0.5 * (lo + hi)
                lo, hi = (mid, hi) if (f(mid) > 0) == s else (lo, mid)
            om.append(0.5 * (lo + hi))
        om = np.array(om)
        lam = 2.0 * c / (om * om + c * c)
        t = np.stack(np.meshgrid(*[np.arange(kmax)] * 3, indexing="ij"), -1).reshape(-1, 3)
        st = np.sort(t, axis=1)
        prod = (lam[st[:, 0]] * lam[st[:, 1]]) * lam[st[:, 2]]
        order = np.lexsort((t[:, 2], t[:, 1], t[:, 0], -prod))
        if len(order) >= M and lam[0] * lam[0] * lam[kmax] < prod[order[M - 1]]:
            break
        kmax *= 2
    pick = order[:M]
    return t[pick], np.sqrt(sigma2 * prod[pick]), om


def _kappa(n, c, xi):
    """exp of the truncated KLE at the element centroids, [B, n(z), n(y), n(x)]."""
    tri, sq, om = _modes(c["corr"], c["sigma2"], c["M"])
    K = int(tri.max()) + 1
    s = (np.arange(n) + 0.5) / n - 0.5
    tab = np.stack([np.cos(om[q] * s) / math.sqrt(0.5 + math.sin(om[q]) / (2 * om[q])) if q % 2 == 0 else
                    np.sin(om[q] * s) / math.sqrt(0.5 - math.sin(om[q]) / (2 * om[q])) for q in range(K)], 1)
    tab = torch.from_numpy(tab).to(xi.device)
    co = torch.zeros((xi.shape[0], K, K, K), dtype=torch.float64, device=xi.device)
    t = torch.from_numpy(tri).to(xi.device)
    co[:, t[:, 2], t[:, 1], t[:, 0]] = xi * torch.from_numpy(sq).to(xi.device)
    g = co @ tab.T                                                    # z y X
    g = (g.transpose(2, 3) @ tab.T).transpose(2, 3)                   # z Y X
    g = (g.permute(0, 2, 3, 1) @ tab.T).permute(0, 3, 1, 2)
    return torch.exp(g)


def _philox_normals(seed, level, ids, M, stream=0):
    """Philox4x64-10, key (seed, 0), counter (sample, level, block, stream); Box-Muller."""
    nb = (M + 3) // 4
    m32 = np.uint64(0xFFFFFFFF)

    def mulhilo(a, b):
        al, ah, bl, bh = a & m32, a >> np.uint64(32), b & m32, b >> np.uint64(32)
        ll, lh, hl = al * bl, al * bh, ah * bl
        mid = (ll >> np.uint64(32)) + (lh & m32) + (hl & m32)
        return ah * bh + (lh >> np.uint64(32)) + (hl >> np.uint64(32)) + (mid >> np.uint64(32)), a * b

    with np.errstate(over="ignore"):
        shape = (len(ids), nb)
        x = [np.broadcast_to(np.asarray(ids, dtype=np.uint64)[:, None], shape).copy(),
             np.broadcast_to(np.asarray(level, dtype=np.uint64).reshape(-1, 1), shape).copy(),
             np.broadcast_to(np.arange(nb, dtype=np.uint64)[None, :], shape).copy(),
             np.full(shape, stream, dtype=np.uint64)]
        k0, k1 = np.uint64(seed), np.uint64(0)
        for r in range(10):
            if r:
                k0, k1 = k0 + np.uint64(0x9E3779B97F4A7C15), k1 + np.uint64(0xBB67AE8584CAA73B)
            h0, l0 = mulhilo(np.full(shape, 0xD2E7470EE14C6C93, dtype=np.uint64), x[0])
            h1, l1 = mulhilo(np.full(shape, 0xCA5A826395121157, dtype=np.uint64), x[2])
            x = [h1 ^ x[1] ^ k0, l1, h0 ^ x[3] ^ k1, l0]
        u = [((w >> np.uint64(12)).astype(np.float64) + 0.5) * 2.0 ** -52 for w in x]
    z = []
    for a, b in ((u[0], u[1]), (u[2], u[3])):
        r = np.sqrt(-2.0 * np.log(a))
        z += [r * np.cos(2 * math.pi * b), r * np.sin(2 * math.pi * b)]
    return np.stack(z, -1).reshape(len(ids), 4 * nb)[:, :M]


_CORNERS = [(dz, dy, dx) for dz in (0, 1) for dy in (0, 1) for dx in (0, 1)]


def _khat(device):
    d = torch.tensor([[sum(p != q for p, q in zip(a, b)) for b in _CORNERS] for a in _CORNERS], device=device)
    k = torch.full((8, 8), -1.0 / 12, dtype=torch.float64, device=device)
    k[d == 0] = 1.0 / 3
    k[d == 1] = 0.0
    return k


def _corner_sum(parts, n):
    """Interior sums [B, n-1, n-1, n-1] of one value per element corner (corner order _CORNERS)."""
    p = parts[0]
    full = torch.zeros((p.shape[0], n + 1, n + 1, n + 1), dtype=p.dtype, device=p.device)
    for v, (dz, dy, dx) in zip(parts, _CORNERS):
        full[:, dz:dz + n, dy:dy + n, dx:dx + n] += v
    return full[:, 1:n, 1:n, 1:n]


def _apply(kap, u, kh):
    n = kap.shape[1]
    up = torch.nn.functional.pad(u, (1, 1, 1, 1, 1, 1))
    c = [up[:, dz:dz + n, dy:dy + n, dx:dx + n] for dz, dy, dx in _CORNERS]
    tot = sum(c)
    parts = []
    for a in range(8):
        # row a of the element matrix: 1/3 on a, 0 on edge neighbours, -1/12 on the others
        near = sum(c[b] for b in range(8) if kh[a][b] == 0.0)
        parts.append(kap * ((1.0 / 3 + 1.0 / 12) * c[a] - (tot - near) / 12))
    return _corner_sum(parts, n) / n


def _diag(kap):
    return _corner_sum([kap] * 8, kap.shape[1]) / (3.0 * kap.shape[1])


def _solve(kap, b, tol=1e-13):
    n = kap.shape[1]
    kh = _khat("cpu").tolist()
    dinv = 1.0 / _diag(kap)
    dot = lambda p, q: (p * q).sum((1, 2, 3), keepdim=True)   # noqa: E731
    x, r = torch.zeros_like(b), b.clone()
    z = dinv * r
    p, rz, bb = z.clone(), dot(r, z), dot(b, b)
    for it in range(40 * n):
        q = _apply(kap, p, kh)
        a = rz / dot(p, q)
        x += a * p
        r -= a * q
        if it % 10 == 9 and bool((dot(r, r) <= tol * tol * bb).all()):
            break
        z = dinv * r
        new = dot(r, z)
        p = z + (new / rz) * p
        rz = new
    return x


def _qoi(u, qoi):
    n = u.shape[1] + 1
    w = torch.ones(n - 1, dtype=torch.float64, device=u.device)
    if qoi == 1:
        i = torch.arange(1, n, device=u.device)
        w = (2.0 * ((i > n // 4) & (i < 3 * n // 4)) + 1.0 * ((i == n // 4) | (i == 3 * n // 4))).double()
    return torch.einsum("bzyx,z,y,x->b", u, w, w, w) / n ** 3


def _qois(c, seed, level, ids, n):
    out = []
    chunk = max(1, (1 << 25) // n ** 3)
    for k in range(0, len(ids), chunk):
        part = ids[k:k + chunk]
        xi = _philox_normals(workloads.DEFAULT_SEED + seed, level, part, c["M"])
        kap = _kappa(n, c, torch.from_numpy(xi).cuda())
        if c["forcing"]:
            xif = _philox_normals(workloads.DEFAULT_SEED + seed, level, part, c["M"], 2)
            b = _corner_sum([_kappa(n, c, torch.from_numpy(xif).cuda())] * 8, n) / (8.0 * n ** 3)
        else:
            b = torch.full((len(part), n - 1, n - 1, n - 1), 1.0 / n ** 3, dtype=torch.float64, device="cuda")
        out.append(_qoi(_solve(kap, b), c["qoi"]))
    return torch.cat(out).cpu().numpy()


def _pairs(c, seed, level, ids):
    qf = _qois(c, seed, level, ids, c["n0"] << level)
    qc = _qois(c, seed, level, ids, c["n0"] << (level - 1)) if level else np.zeros(len(ids))
    return qf - qc, qf, qc


def _to_grid(v, n):
    """Interior values [B, n-1, n-1, n-1] in the library's grid layout (i + n j + n^2 k, zero boundary)."""
    full = torch.zeros((v.shape[0], n + 1, n, n), dtype=v.dtype, device=v.device)
    full[:, 1:n, 1:, 1:] = v
    full = full.reshape(v.shape[0], -1)
    return torch.nn.functional.pad(full, (0, mm.grid_stride(n) - full.shape[1]))


def _prolong(n):
    """1D trilinear prolongation from the n/2 grid's interior nodes to the n grid's."""
    P = torch.zeros((n - 1, n // 2 - 1), dtype=torch.float64, device="cuda")
    for J in range(1, n // 2):
        P[2 * J - 1, J - 1] = 1.0
        P[2 * J - 2, J - 1] = P[2 * J, J - 1] = 0.5
    return P


def _axes(M, v):
    for _ in range(3):
        v = (v @ M.T).permute(0, 3, 1, 2)   # the last axis, then the one before it, ...
    return v


def _vcycle(kap, b, deg):
    n = kap.shape[1]
    if n == 2:
        return b / _diag(kap)
    kh = _khat("cpu").tolist()
    dinv = 1.0 / _diag(kap)
    theta, delta = 0.5 * (1.75 + 0.4375), 0.5 * (1.75 - 0.4375)

    def smooth(x, zero):
        rho, prev = delta / theta, x
        x = prev + (dinv * (b if zero else b - _apply(kap, prev, kh))) / theta
        first = prev
        for _ in range(1, deg):
            nrho = 1.0 / (2.0 * theta / delta - rho)
            x, first = x + nrho * rho * (x - first) + 2.0 * nrho / delta * dinv * (b - _apply(kap, x, kh)), x
            rho = nrho
        return x

    x = smooth(torch.zeros_like(b), True)
    P = _prolong(n)
    B, m = kap.shape[0], n // 2
    kc = kap.reshape(B, m, 2, m, 2, m, 2).mean((2, 4, 6))
    xc = _vcycle(kc, _axes(P.T, b - _apply(kap, x, kh)), deg)
    return smooth(x + _axes(P, xc), False)


def exact(case, seed):
    c = _full(case)
    n, kind = c["n0"] << c["level"], c["kind"]
    if kind == "field":
        if c["count"] * n ** 3 > 1 << 26:
            return None
        k = _kappa(n, c, _xi(c, seed).cuda()).reshape(c["count"], -1)
        return {"kappa": k, "kappa32": k}
    # Jacobi-PCG takes ~4 n iterations: what that costs decides whether there is a value
    total = {"estimate": 262, "serve": c["count"]}.get(kind, c["count"])
    if (n > 128 or total * n ** 3 > 1 << 25) and kind != "vcycle":
        return None
    ids = np.arange(c["count"], dtype=np.uint64) + np.uint64(_first(seed))
    if kind == "sample":
        y, qf, qc = _pairs(c, seed, c["level"], ids)
        return {"y": y, "q_fine": qf, "q_coarse": qc}
    if kind == "serve":
        lv = _serve_levels(c, seed)
        out = np.zeros((3, c["count"]))
        for l in range(c["levels"]):
            out[:, lv == l] = _pairs(c, seed, l, ids[lv == l])
        return {"y": out[0], "q_fine": out[1], "q_coarse": out[2]}
    if kind == "estimate":
        ns = [int(x) for x in c["n_fixed"].split(",")]
        ys = [_pairs(c, seed, l, np.arange(k, dtype=np.uint64))[0] for l, k in enumerate(ns)]
        m2 = np.array([((y - y.mean()) ** 2).sum() for y in ys])
        return {"qtilde": float(sum(y.mean() for y in ys)), "var": float(sum(v / k / k for v, k in zip(m2, ns))),
                "n": np.array(ns), "mean": np.array([y.mean() for y in ys]), "m2": m2}
    kap = _kappa(n, c, _xi(c, seed).cuda())
    if kind == "solve":
        b = torch.full((c["count"], n - 1, n - 1, n - 1), 1.0 / n ** 3, dtype=torch.float64, device="cuda")
        return {"u": _to_grid(_solve(kap, b), n), "iters": None}
    dt = torch.float64 if c["precision"] == 0 else torch.float32
    r = _rhs(c, seed, dt).double().reshape(c["count"], n - 1, n - 1, n - 1)
    return {"z": _to_grid(_vcycle(kap.to(dt).double(), r, c["degree"] or 2), n)}
