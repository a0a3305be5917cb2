"""Performance cases: windows that a user solves through ``solve`` (and
``solve_noalloc``), over the range of sizes, dimensions, paths and options the
library supports. Inputs are synthetic, shaped like the recipes of
``paper_2607_24741_amd.workloads`` (toy clouds, mixtures, telemetry, features,
LiDAR), drawn on the GPU from a seed.

A case is a dict of plain values:
  kind       recipe of the points, masses and eps
  W, n, m, d window width, points per side (padded size when ``ragged``), dimension
  ragged     lanes of different sizes (n_t ~ U{n/32..n}, m_t ~ U{m/32..m})
  tol, max_iter, audit_every, mode
  path       "default", "fast32", "matrix_free", "guard" (the flags of the call)
  warm       start from the solution of a slightly earlier frame (streaming)
  noalloc    call ``solve_noalloc`` with caller-owned outputs
  cycles     cycles a lane typically needs (for work() only)
"""

from __future__ import annotations

import math

import torch

import paper_2607_24741_amd as ds

DEV = "cuda:0"
FLAGS = {"default": 0, "fast32": ds.F_FAST32, "matrix_free": ds.F_MATRIX_FREE, "guard": ds.F_GUARD}


def _case(name, kind, W, n, m, d, *, cycles, tol=1e-3, max_iter=5000, audit_every=1, mode="active",
          path="default", ragged=False, warm=False, noalloc=False):
    c = dict(kind=kind, W=W, n=n, m=m, d=d, cycles=cycles, tol=tol, max_iter=max_iter,
             audit_every=audit_every, mode=mode, path=path, ragged=ragged, warm=warm,
             noalloc=noalloc)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the toy window of the tests and the benchmark: a thousand cycles of tiny
        # lanes, where latency and launches are all there is
        _case("toy", "toy", 8, 64, 64, 2, cycles=330),
        # a small streaming call: consecutive frames, each started from the one
        # before, without allocation in the call
        _case("warm_frames", "lidar", 12, 300, 257, 3, cycles=60, warm=True, noalloc=True),
        # the mixture window of the benchmark (single-cell shaped): a long narrow tail
        _case("mixture", "mixture", 64, 1024, 1024, 8, cycles=2700),
        # the telemetry window: many lanes, d = 16
        _case("telemetry", "telemetry", 256, 512, 512, 16, cycles=3400),
        # the headline LiDAR window: lanes of 256 to 8192 points
        _case("lidar", "lidar", 1024, 8192, 8192, 3, cycles=224, ragged=True),
        # one large scan pair on its own: the chip has to be filled from one lane
        _case("one_scan", "lidar", 1, 8192, 7001, 3, cycles=300),
        # feature couplings (d = 512, materialised cost), audited every 4 cycles
        _case("features", "features", 16, 4096, 4096, 512, cycles=500, audit_every=4),
        # a pair of sides beyond what the materialised cost takes: matrix-free
        _case("large_sides", "features", 1, 18001, 16500, 64, cycles=40, tol=1e-6, max_iter=40),
        # reduced feature space (16 < d <= 32): float32 matrix-core path, fixed budget
        _case("reduced_features", "mixture", 32, 768, 700, 24, cycles=300, tol=1e-7, max_iter=300),
        # the opt-in float32 state, fixed budget
        _case("fast32_budget", "mixture", 32, 1024, 1024, 8, cycles=300, tol=1e-7, max_iter=300,
              path="fast32"),
        # certified release of telemetry windows
        _case("guarded", "telemetry", 32, 512, 500, 16, cycles=3400, path="guard", audit_every=4),
        # static packing of a small odd window
        _case("static", "mixture", 16, 513, 700, 5, cycles=2000, mode="static", tol=3e-3),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more window of the ranges above. Windows of the paths with a float32
    state run a fixed budget of cycles, the others to their tolerance."""
    kind = rng.choice(["toy", "warm", "mixture", "telemetry", "lidar", "features", "reduced",
                       "fast32", "guard", "large"])
    if kind == "toy":
        return _case(None, "toy", _log_int(rng, 1, 128), _log_int(rng, 16, 256),
                     _log_int(rng, 16, 256), rng.randint(1, 4), cycles=330,
                     audit_every=rng.choice([1, 1, 4]))
    if kind == "warm":
        return _case(None, "lidar", _log_int(rng, 1, 32), _log_int(rng, 64, 1024),
                     _log_int(rng, 64, 1024), rng.choice([2, 3]), cycles=60, warm=True,
                     noalloc=rng.random() < 0.5)
    if kind == "mixture":
        return _case(None, "mixture", _log_int(rng, 1, 64), _log_int(rng, 128, 1024),
                     _log_int(rng, 128, 1024), rng.randint(4, 12), cycles=2000,
                     mode=rng.choice(["active", "active", "static", "logical"]),
                     tol=rng.choice([1e-2, 3e-3, 1e-3]))
    if kind == "telemetry":
        return _case(None, "telemetry", _log_int(rng, 4, 256), _log_int(rng, 64, 512),
                     _log_int(rng, 64, 512), rng.randint(9, 16), cycles=3000,
                     audit_every=rng.choice([1, 4]))
    if kind == "lidar":
        return _case(None, "lidar", _log_int(rng, 1, 256), _log_int(rng, 512, 8192),
                     _log_int(rng, 512, 8192), 3, cycles=224, ragged=rng.random() < 0.7)
    if kind == "features":
        return _case(None, "features", _log_int(rng, 1, 12), _log_int(rng, 256, 4096),
                     _log_int(rng, 256, 4096), rng.randint(33, 512), cycles=300, audit_every=4,
                     tol=1e-6, max_iter=300)
    if kind == "reduced":
        return _case(None, "mixture", _log_int(rng, 1, 64), _log_int(rng, 128, 1024),
                     _log_int(rng, 128, 1024), rng.randint(17, 32), cycles=300, tol=1e-7,
                     max_iter=300)
    if kind == "fast32":
        return _case(None, "mixture", _log_int(rng, 1, 64), _log_int(rng, 128, 1024),
                     _log_int(rng, 128, 1024), rng.randint(2, 16), cycles=300, tol=1e-7,
                     max_iter=300, path="fast32")
    if kind == "guard":
        return _case(None, "telemetry", _log_int(rng, 4, 64), _log_int(rng, 64, 512),
                     _log_int(rng, 64, 512), rng.randint(8, 16), cycles=3000, path="guard",
                     audit_every=4)
    return _case(None, "features", 1, _log_int(rng, 1024, 18000), _log_int(rng, 1024, 18000),
                 rng.randint(33, 128), cycles=40, tol=1e-6, max_iter=40, path="matrix_free")


# ------------------------------------------------------------------ inputs
def _unit(v):
    return v / v.norm(dim=-1, keepdim=True)


def _inputs(case, seed):
    """float32 X, Y, a, b, eps and int32 n, m of a window, float64-normalised."""
    W, n, m, d, kind = case["W"], case["n"], case["m"], case["d"], case["kind"]
    gen = torch.Generator(device=DEV)
    gen.manual_seed(1_000_003 * seed + 17)
    f64 = dict(dtype=torch.float64, device=DEV, generator=gen)
    randn = lambda *s: torch.randn(*s, **f64)
    rand = lambda *s: torch.rand(*s, **f64)
    nt = torch.full((W,), n, dtype=torch.int64, device=DEV)
    mt = torch.full((W,), m, dtype=torch.int64, device=DEV)
    if case["ragged"]:
        nt = (n // 32 + (rand(W) * (n - n // 32 + 1)).long()).clamp(1, n)
        mt = (m // 32 + (rand(W) * (m - m // 32 + 1)).long()).clamp(1, m)
    uniform = False
    if kind == "toy":
        # Gaussian clouds, target shifted by U(0, 1)^d, eps ~ logU(0.02, 0.2)
        X, Y = randn(W, n, d), randn(W, m, d) + rand(W, 1, d)
        eps = torch.exp(math.log(0.02) + math.log(10.0) * rand(W))
        uniform = True
    elif kind == "mixture":
        # 4-component mixtures, Dirichlet(1) masses; eps 0.05 at d = 8, in
        # proportion to d (the mean cost is)
        def cloud(k):
            mu = 2.0 * randn(W, 4, d)
            comp = (rand(W, k) * 4).long().clamp(max=3)
            return torch.gather(mu, 1, comp[:, :, None].expand(W, k, d)) + 0.5 * randn(W, k, d)
        X, Y = cloud(n), cloud(m)
        a, b = -torch.log1p(-rand(W, n)), -torch.log1p(-rand(W, m))
        eps = torch.full((W,), 0.05 * max(1.0, d / 8.0), dtype=torch.float64, device=DEV)
    elif kind == "telemetry":
        # AR(1) channels: a window, a gap and a shifted later window; eps 0.01
        phi = 0.5 + 0.49 * rand(W, 1)
        gap, burn = 512, 200
        z = randn(burn + n + gap + m, W, d) * torch.sqrt(1.0 - phi * phi)
        s = [randn(W, d)]
        for k in range(1, burn + n + gap + m):
            s.append(phi * s[-1] + z[k])
        s = torch.stack(s, 1)
        X = s[:, burn:burn + n]
        Y = s[:, burn + n + gap:] + (0.5 + 1.5 * rand(W, 1, 1)) * _unit(randn(W, 1, d))
        eps = torch.full((W,), 0.01, dtype=torch.float64, device=DEV)
        uniform = True
    elif kind == "features":
        # unit features around 10 class means, E cos = 0.7; eps 0.05
        means = _unit(randn(W, 10, d))
        sigma = math.sqrt((0.7 ** -2 - 1.0) / d)

        def feats(k):
            lab = (rand(W, k) * 10).long().clamp(max=9)
            return _unit(torch.gather(means, 1, lab[:, :, None].expand(W, k, d))
                         + sigma * randn(W, k, d))
        X, Y = feats(n), feats(m)
        eps = torch.full((W,), 0.05, dtype=torch.float64, device=DEV)
        uniform = True
    else:
        # a cube against a noisy sphere, Dirichlet(0.5) masses, eps ~ logU(0.005, 0.1)
        X = 2.0 * rand(W, n, d) - 1.0
        Y = _unit(randn(W, m, d)) + 0.02 * randn(W, m, d)
        a, b = randn(W, n) ** 2, randn(W, m) ** 2
        eps = torch.exp(math.log(0.005) + math.log(20.0) * rand(W))
    inx = torch.arange(n, device=DEV)[None, :] < nt[:, None]
    iny = torch.arange(m, device=DEV)[None, :] < mt[:, None]
    if uniform:
        a, b = torch.ones(W, n, dtype=torch.float64, device=DEV), torch.ones(W, m, dtype=torch.float64, device=DEV)
    a, b = a * inx, b * iny
    a, b = a / a.sum(1, keepdim=True), b / b.sum(1, keepdim=True)
    f = lambda t: t.to(torch.float32).contiguous()
    return dict(X=f(X * inx[:, :, None]), Y=f(Y * iny[:, :, None]), a=f(a), b=f(b), eps=f(eps),
                n=nt.to(torch.int32), m=mt.to(torch.int32))


def prepare(case, seed):
    s = _inputs(case, seed)
    kw = dict(max_iter=case["max_iter"], audit_every=case["audit_every"], mode=case["mode"],
              flags=FLAGS[case["path"]])
    if case["warm"]:
        # the previous frame: the same scan a small motion earlier, and its solution
        gen = torch.Generator(device=DEV)
        gen.manual_seed(7_000_003 * seed + 5)
        prev = s["Y"] + 0.01 * torch.randn(s["Y"].shape, dtype=torch.float32, device=DEV, generator=gen)
        kw["g0"] = ds.solve(s["X"], prev, s["a"], s["b"], s["eps"], case["tol"], n=s["n"], m=s["m"],
                            max_iter=case["max_iter"])[1]
    if case["noalloc"]:
        W = case["W"]
        f32, i32 = dict(dtype=torch.float32, device=DEV), dict(dtype=torch.int32, device=DEV)
        kw["out"] = dict(f=torch.empty(W, case["n"], **f32), g=torch.empty(W, case["m"], **f32),
                         depth=torch.empty(W, **i32), residual=torch.empty(W, **f32),
                         status=torch.empty(W, **i32))
    return dict(s, tol=case["tol"], kw=kw, noalloc=case["noalloc"])


def run(state):
    s = state
    call = ds.solve_noalloc if s["noalloc"] else ds.solve
    out = call(s["X"], s["Y"], s["a"], s["b"], s["eps"], s["tol"], n=s["n"], m=s["m"], **s["kw"])
    return dict(f=out[0], g=out[1], depth=out[2], residual=out[3], status=out[4])


# ------------------------------------------------------ work and tolerances
def _terms(case):
    """(i, j) pairs of the window (ragged lanes: the mean of the product)."""
    share = (0.5 * (1.0 + 1.0 / 32.0)) ** 2 if case["ragged"] else 1.0
    return case["W"] * case["n"] * case["m"] * share


def work(case):
    """Inputs read once, outputs written once; per pair and half-step an
    exponential with its add and scale, and the d multiply-adds of the exponent
    -- once per solve where the window's costs can be kept (d > 32 and up to
    16384 points a side, unless the call asks for the matrix-free path)."""
    W, n, m, d = case["W"], case["n"], case["m"], case["d"]
    share = 0.5 * (1.0 + 1.0 / 32.0) if case["ragged"] else 1.0
    bytes_ = 4.0 * W * share * (n * (d + 2) + m * (d + 2 + (1 if case["warm"] else 0))) + 24.0 * W
    kept = d > 32 and max(n, m) <= 16384 and case["path"] != "matrix_free"
    halves = 2.0 * min(case["cycles"], case["max_iter"])
    flops = _terms(case) * (2.0 * d * (1.0 if kept else halves) + 4.0 * halves)
    return dict(bytes=bytes_, flops=flops)


def tolerance(case):
    """Float64 state: potentials to their float32 rounding, residuals to about
    1e-8 of a tolerance of 1e-3. Float32 states: the rounding of coordinates,
    costs and potentials moves exponents of size cost / eps. A few lanes in a
    thousand sit near enough to the tolerance to stop a cycle earlier or later."""
    if case["d"] > 16 or case["path"] in ("fast32", "matrix_free"):
        return dict(rel=2e-3, max=2e-2, differ=0.005)
    return dict(rel=1e-4, max=1e-2, differ=0.005)


# -------------------------------------------------------------- reference
def exact(case, seed):
    """The same windows in float64 with torch alone: dense kernels
    K = exp((F + G - C) / eps) around absorbed potentials (F, G), scalings u, v,
    re-absorbed when they grow; the first cycles in the log domain."""
    if case["path"] == "guard" or _terms(case) * case["cycles"] > 3e12 or _terms(case) > 1e9:
        return None
    state = prepare(case, seed)
    t64 = lambda k: state[k].to(torch.float64)
    X, Y, a, b, eps = t64("X"), t64("Y"), t64("a"), t64("b"), t64("eps")
    W, n, m = case["W"], case["n"], case["m"]
    tol, ae, max_iter = float(case["tol"]), case["audit_every"], case["max_iter"]
    C = torch.empty(W, n, m, dtype=torch.float64, device=DEV)
    for t in range(W):
        c = 0.5 * (X[t].mean(0) + Y[t].mean(0))
        x, y = X[t] - c, Y[t] - c
        if case["d"] <= 16:
            C[t] = 0.0
            for k in range(case["d"]):
                C[t] += (x[:, k, None] - y[None, :, k]) ** 2
        else:
            C[t] = ((x * x).sum(1)[:, None] + (y * y).sum(1)[None, :] - 2.0 * (x @ y.T)).clamp(min=0)
    la, lb = torch.log(a), torch.log(b)     # -inf at padding and zero masses
    e1 = eps[:, None]
    g0 = state["kw"].get("g0")
    G = torch.zeros(W, m, dtype=torch.float64, device=DEV) if g0 is None else g0.to(torch.float64)
    G = torch.where(b > 0, G, torch.full_like(G, -math.inf))
    F = torch.full((W, n), -math.inf, dtype=torch.float64, device=DEV)
    ids = torch.arange(W, device=DEV)
    out = dict(f=torch.zeros(W, n, dtype=torch.float64, device=DEV),
               g=torch.zeros(W, m, dtype=torch.float64, device=DEV),
               depth=torch.zeros(W, dtype=torch.int32, device=DEV),
               residual=torch.zeros(W, dtype=torch.float64, device=DEV),
               status=torch.ones(W, dtype=torch.int32, device=DEV))
    static = case["mode"] == "static"
    passed = torch.zeros(W, dtype=torch.bool, device=DEV)

    def lse(v, dim):
        # log sum exp of (v - C) / eps over dim, a lane at a time to bound memory
        parts = []
        for q in range(len(ids)):
            z = (v[q][None, :] if dim == 1 else v[q][:, None]) - C[q]
            parts.append(torch.logsumexp(z / eps[q], dim=dim))
        return torch.stack(parts)

    def kernel():
        K = torch.empty_like(C)
        for q in range(len(ids)):
            torch.exp((F[q][:, None] + G[q][None, :] - C[q]) / eps[q], out=K[q])
        return K

    Fin = lambda v: torch.where(torch.isfinite(v), v, torch.zeros_like(v))
    K = u = v = None
    for k in range(1, max_iter + 1):
        if k <= 4:
            F = eps[:, None] * (la - lse(G, 1))
            G = eps[:, None] * (lb - lse(F, 0))
            K = None
        else:
            if K is None:
                K = kernel()
                u, v = torch.ones_like(a), torch.ones_like(b)
            s = torch.bmm(K, v[:, :, None])[:, :, 0]
            u = torch.where(a > 0, a / s, torch.zeros_like(a))
            s = torch.bmm(u[:, None, :], K)[:, 0, :]
            v = torch.where(b > 0, b / s, torch.zeros_like(b))
        if k % ae and k != max_iter:
            continue
        if k <= 4:
            Kk = kernel()
            R, Cm = Kk.sum(2), Kk.sum(1)
            del Kk
        else:
            R, Cm = u * torch.bmm(K, v[:, :, None])[:, :, 0], v * s
        res = torch.maximum((R - a).abs().sum(1), (Cm - b).abs().sum(1))
        ok = res <= tol
        # (static packing: every lane runs on until the last has passed)
        first = ok & ~passed
        if static:
            out["depth"][ids[first]] = k
            out["status"][ids[first]] = 0
            passed |= ok
            end = bool(passed.all()) or k == max_iter
            stop = torch.full_like(ok, end)
        else:
            stop = ok | (k == max_iter)
        if bool(stop.any()):
            f = F if K is None else F + e1 * torch.log(u)
            g = G if K is None else G + e1 * torch.log(v)
            sel = ids[stop]
            out["f"][sel], out["g"][sel] = Fin(f[stop]), Fin(g[stop])
            out["residual"][sel] = res[stop]
            if static:
                out["depth"][ids[~passed]] = k
            else:
                out["depth"][sel] = k
                out["status"][sel] = torch.where(ok[stop], 0, 1).to(torch.int32)
            live = ~stop
            if not bool(live.any()):
                break
            ids, C, F, G, a, b = ids[live], C[live], F[live], G[live], a[live], b[live]
            la, lb, eps, e1, passed = la[live], lb[live], eps[live], e1[live], passed[live]
            if K is not None:
                K, u, v = K[live], u[live], v[live]
        if K is not None and k % 8 == 0:
            grow = torch.maximum(torch.log(u[a > 0]).abs().max(), torch.log(v[b > 0]).abs().max())
            if float(grow) > 40.0:
                F, G, K = F + e1 * torch.log(u), G + e1 * torch.log(v), None
    return dict(f=out["f"], g=out["g"], depth=None, residual=out["residual"], status=None)
