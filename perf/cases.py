"""The work users have this library do, as cases that can be timed and compared.

Every case is one call (or a forward and its backward) through the public
entry points ``Solver.solve`` and ``Solver.adjoint`` on a synthetic book of
one of the shapes the repository's workloads, tests and benchmark use.  The
data follows the same distributions as ``workloads.books`` but is drawn on
the GPU, so that a book of 500 x 10,000 takes milliseconds to make.

A case's fields:
  m, n, k     accounts, assets, factors
  groups      sector bands (0: none) of half-width ``band``
  halves      policy halfspace rows (factor exposures within 5e-3)
  ub, gamma, kappa   box [0, ub], risk aversion, L1 trade cost
  held        0: dense drifted holdings, else about this many held names
  tax         4-lot piecewise-linear tax on the sales of the held names
  excl        exclusion masks leaving U[0.3, 1] of the names eligible
  cap         turnover cap at the least feasible turnover + 0.1
  bounds      per-asset bounds and minimum holdings
  bench       benchmark-relative risk and a return scale per account
  rho, alpha, check, first, rounds, precision   the solver's schedule
  eps         residual tolerance (1e-9 where gradients are wanted: they belong to the pattern of
              the optimum itself, and a pattern accepted at 1e-6 can move them by a percent)
  mode        "solve", "warm" (from the state of the day before, returning
              the new state), "grad" (forward + KKT adjoint), "adjoint" (the
              backward alone, after a solve the program already has)

``run`` returns what the program acts on: the float64 weights, the objective
and the status (and the gradients / the state where the mode has them).  The
multipliers are not unique at degenerate patterns and the residuals are
rounding noise around zero, so neither has a value to compare.
"""
import math

import torch

from paper_2606_23367_amd.solver import DeviceProblem, Solver

_BASE = dict(m=1, n=100, k=5, groups=0, band=0.05, halves=0, ub=0.1, gamma=1.0, kappa=0.0,
             held=0, tax=False, excl=False, cap=False, bounds=False, bench=False,
             rho=1.0, alpha=1.6, check=50, first=0, rounds=16, precision=1,
             eps=1e-6, mode="solve")


def _case(name, **over):
    return dict(_BASE, name=name, **over)


def listed():
    return [
        # one small account, interactive: latency and launches are everything
        _case("one account 100", rho=0.05),
        # the small-universe batch: 200 accounts on 481 names, L1 transition cost
        _case("batch 200x481", m=200, n=481, k=20, ub=0.03, kappa=5e-3, rho=1.0, alpha=1.8),
        # a what-if on one account of the large book: one account per call,
        # float32 contractions
        _case("one account 10000 fp32", n=10000, k=80, ub=0.01, held=250, tax=True, excl=True,
              cap=True, rho=10.0, alpha=1.8, precision=0),
        # a mid-size book with sector bands
        _case("bands 64x2000", m=64, n=2000, k=40, groups=10, ub=0.05, kappa=1e-3, rho=1.0,
              alpha=1.8),
        # the same size with every rule family: bands, halfspaces, exclusions, tax lots
        _case("rules 64x2000", m=64, n=2000, k=40, groups=10, halves=5, ub=0.05, kappa=1e-3,
              held=400, tax=True, excl=True, rho=1.0, alpha=1.8),
        # the rest of the problem class: per-asset bounds, benchmark, return scale
        _case("benchmark 37x3001", m=37, n=3001, k=33, groups=10, ub=0.02, kappa=1e-3,
              gamma=100.0, bounds=True, bench=True, rho=1.0),
        # differentiation through a risk-averse book: forward and backward
        _case("grad 128x5000", m=128, n=5000, k=60, groups=10, ub=0.02, gamma=1000.0, kappa=1e-3,
              rho=1.0, eps=1e-9, mode="grad"),
        # the backward alone
        _case("adjoint 128x5000", m=128, n=5000, k=60, groups=10, ub=0.02, kappa=1e-3, rho=1.0,
              eps=1e-9, mode="adjoint"),
        # the production queue: 500 accounts, exclusions, taxed holdings, turnover cap
        _case("queue 500x10000", m=500, n=10000, k=80, ub=0.01, held=250, tax=True, excl=True,
              cap=True, rho=10.0, alpha=1.8, first=150, rounds=24),
        # the same queue the next day, from the stored state
        _case("warm 500x10000", m=500, n=10000, k=80, ub=0.01, held=250, tax=True, excl=True,
              cap=True, rho=10.0, alpha=1.8, first=50, rounds=24, mode="warm"),
        # a very wide universe: 8 accounts, 50 groups, taxed holdings
        _case("wide 8x384800", m=8, n=384800, k=100, groups=50, band=0.005, ub=1e-3, kappa=1e-3,
              held=2000, tax=True, rho=10.0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("plain", "bands", "rules", "queue", "queue", "grad", "adjoint", "wide"))
    c = dict(_BASE)
    if kind == "plain":
        n = _log(rng, 100, 1000)
        c.update(m=_log(rng, 1, 300), n=n, k=rng.randint(5, 24), ub=max(0.03, 10.0 / n),
                 kappa=5e-3, rho=1.0, alpha=1.8)
    elif kind in ("bands", "rules"):
        n = _log(rng, 700, 5000)
        c.update(m=_log(rng, 4, 128), n=n, k=rng.randint(10, 60), groups=10,
                 ub=max(0.02, 50.0 / n), kappa=1e-3, rho=1.0, alpha=1.8)
        if kind == "rules":
            c.update(halves=5, held=400, tax=True, excl=True)
    elif kind == "queue":
        n = _log(rng, 1300, 16000)
        c.update(m=_log(rng, 1, 500), n=n, k=rng.randint(8, 95), ub=0.01,
                 held=rng.randint(100, 300), tax=True, excl=True, cap=True, rho=10.0, alpha=1.8,
                 first=rng.choice((0, 100, 150)), rounds=24)
        while c["m"] * c["n"] > 5_000_000:
            c["m"] = max(1, c["m"] // 2)
    elif kind in ("grad", "adjoint"):
        c.update(m=_log(rng, 4, 128), n=_log(rng, 900, 5000), k=rng.randint(12, 60), groups=10,
                 ub=0.02, gamma=rng.choice((1.0, 1000.0)), kappa=1e-3, rho=1.0, eps=1e-9,
                 mode=kind)
    else:
        c.update(m=rng.randint(1, 8), n=_log(rng, 20000, 200000), k=rng.randint(60, 110),
                 groups=rng.choice((40, 50)), band=0.005, ub=1e-3, kappa=1e-3, held=2000,
                 tax=True, rho=10.0)
    return c


def _project(v, cap):
    """Row-wise Euclidean projection onto {0 <= x <= cap, sum x = 1} (cap [m, 1])."""
    lo, hi = v.min(1, keepdim=True)[0] - cap - 1.0, v.max(1, keepdim=True)[0] + 1.0
    for _ in range(60):
        mid = 0.5 * (lo + hi)
        over = torch.minimum((v - mid).clamp_min(0.0), cap).sum(1, keepdim=True) > 1.0
        lo, hi = torch.where(over, mid, lo), torch.where(over, hi, mid)
    return torch.minimum((v - 0.5 * (lo + hi)).clamp_min(0.0), cap)


def _inputs(c, seed):
    """The universe and the book, float32 on the GPU, from the seed alone."""
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed) * 1000003 + 17)
    m, n, k, G, H = c["m"], c["n"], c["k"], c["groups"], c["halves"]
    f64 = dict(dtype=torch.float64, device=dev, generator=g)

    def uniform(lo, hi, *shape):
        return lo + (hi - lo) * torch.rand(*shape, **f64)

    B = (0.1 * torch.randn(n, k, **f64)).float()
    f, d = uniform(0.01, 0.05, k).float(), uniform(1e-4, 1e-3, n).float()
    group = torch.randint(0, G, (n,), device=dev, generator=g, dtype=torch.int32) if G else None
    mu = (5e-4 + 1e-2 * torch.randn(m, n, **f64)).float()
    full = lambda x: torch.full((m,), x, dtype=torch.float32, device=dev)  # noqa: E731
    elig = torch.ones(m, n, dtype=torch.bool, device=dev)
    if c["excl"]:
        frac = uniform(0.3, 1.0, m, 1)
        rank = torch.rand(m, n, **f64).argsort(1).argsort(1)
        elig = rank < torch.ceil(frac * n)
    if c["held"]:
        # 40 % to 160 % of `held` names, never more than half of the universe
        cnt = (uniform(0.4, 1.6, m, 1) * c["held"]).clamp(min(n, 3), max(3, n // 2)).floor()
        rank = torch.rand(m, n, **f64).argsort(1).argsort(1)
        raw = torch.where(rank < cnt, -torch.log(torch.rand(m, n, **f64).clamp_min(1e-300)), -9.0)
        raw = torch.where(rank < cnt, raw / raw.clamp_min(0.0).sum(1, keepdim=True), raw)
        w0 = _project(raw, torch.clamp(1.0 / cnt, min=c["ub"])).float()
    else:
        e = -torch.log(torch.rand(m, n, **f64).clamp_min(1e-300))
        w0 = (e / e.sum(1, keepdim=True)).float()
    tax = (None,) * 4
    if c["tax"]:
        acc, asset = torch.nonzero(w0 > 0, as_tuple=True)
        cnt = torch.bincount(acc, minlength=m)
        ptr = torch.cat([cnt.new_zeros(1), cnt.cumsum(0)]).int()
        fr = -torch.log(torch.rand(acc.numel(), 4, **f64).clamp_min(1e-300))
        brk = ((fr / fr.sum(1, keepdim=True)).cumsum(1)[:, :3] * w0[acc, asset].double()[:, None]).float()
        inf = torch.tensor(math.inf, device=dev)
        for j in (1, 2):
            brk[:, j] = torch.maximum(brk[:, j], torch.nextafter(brk[:, j - 1], inf))
        slope = uniform(0.0, 5e-3, acc.numel(), 4).float().sort(1)[0]
        tax = (ptr, asset.int(), brk.contiguous(), slope.contiguous())
    band_lo = band_hi = half = half_lo = half_hi = lb_a = ub_a = wb = eta = None
    if G:
        share = torch.bincount(group.long(), minlength=G).double() / n
        band_lo = (share - c["band"]).clamp_min(0.0).float().expand(m, G).contiguous()
        band_hi = (share + c["band"]).float().expand(m, G).contiguous()
    if H:
        half = B[:, :H].t().contiguous()
        ew = half.double().mean(1)
        half_lo = (ew - 5e-3).float().expand(m, H).contiguous()
        half_hi = (ew + 5e-3).float().expand(m, H).contiguous()
        half_lo[:, H - 1] = -math.inf
    if c["bounds"]:
        ub_a = (c["ub"] * uniform(0.5, 1.5, m, n)).float()
        lb_a = torch.where((torch.rand(m, n, **f64) < 0.02) & elig, 0.2 * ub_a, torch.zeros_like(ub_a))
    if c["bench"]:
        raw = -torch.log(torch.rand(m, n, **f64).clamp_min(1e-300))
        capb = ub_a.double() if ub_a is not None else torch.full((m, n), c["ub"], **{k2: f64[k2] for k2 in ("dtype", "device")})
        wb = torch.minimum(_project(raw / raw.sum(1, keepdim=True), capb.max(1, keepdim=True)[0]), capb).float()
        eta = uniform(0.5, 1.5, m).float()
    tau = full(math.inf)
    if c["cap"]:
        u = torch.where(elig, torch.tensor(c["ub"], dtype=torch.float64, device=dev), 0.0)
        tau = (2.0 * (w0.double() - u).clamp_min(0.0).sum(1) + 0.1).float()
    words = None
    if c["excl"]:
        W = (n + 31) // 32
        bits = torch.zeros(m, 32 * W, dtype=torch.int64, device=dev)
        bits[:, :n] = elig
        word = (bits.view(m, W, 32) << torch.arange(32, device=dev)).sum(2)
        words = torch.where(word >= 1 << 31, word - (1 << 32), word).int().contiguous()
    return DeviceProblem(
        n=n, k=k, G=G, m=m, B=B, f=f, d=d, group=group, mu=mu, w0=w0, lb=full(0.0),
        ub=full(c["ub"]), eligible=words, gamma=full(c["gamma"]), kappa=full(c["kappa"]), tau=tau,
        band_lo=band_lo, band_hi=band_hi, tax_ptr=tax[0], tax_asset=tax[1], tax_brk=tax[2],
        tax_slope=tax[3], H=H, half=half, half_lo=half_lo, half_hi=half_hi, lb_asset=lb_a,
        ub_asset=ub_a, wb=wb, eta=eta), g


def _settings(c):
    return dict(rho=c["rho"], alpha=c["alpha"], check_every=c["check"], first_check=c["first"],
                polish_rounds=c["rounds"], precision=c["precision"], eps_prim=c["eps"],
                eps_dual=c["eps"], eps_comp=c["eps"])


def prepare(case, seed):
    c = dict(_BASE, **case)
    P, g = _inputs(c, seed)
    s = dict(P=P, solver=Solver(0), mode=c["mode"], settings=_settings(c))
    if c["mode"] in ("grad", "adjoint"):
        s["c"] = torch.randn(c["m"], c["n"], dtype=torch.float64, device="cuda:0", generator=g)
    if c["mode"] == "adjoint":
        s["solver"].solve(P, **s["settings"])
    if c["mode"] == "warm":
        # yesterday's solve left its state; today's returns moved by 1 % of their spread
        first = dict(s["settings"], first_check=150)
        s["state"] = s["solver"].solve(P, want_state=True, **first)["state"]
        P.mu += (1e-4 * torch.randn(P.m, P.n, dtype=torch.float64, device="cuda:0", generator=g)).float()
    return s


def run(s):
    P, solver = s["P"], s["solver"]
    if s["mode"] == "adjoint":
        dmu, dB = solver.adjoint(s["c"])
        return {"dmu": dmu, "dB": dB}
    if s["mode"] == "warm":
        out = solver.solve(P, warm_state=s["state"], want_state=True, warm_start=1, **s["settings"])
        return {"w": out["w"], "obj": out["obj"], "status": out["status"], "state": out["state"]}
    out = solver.solve(P, **s["settings"])
    got = {"w": out["w"], "obj": out["obj"], "status": out["status"]}
    if s["mode"] == "grad":
        got["dmu"], got["dB"] = solver.adjoint(s["c"])
    return got


def work(case):
    c = dict(_BASE, **case)
    m, n, k = c["m"], c["n"], c["k"]
    held = min(c["held"], n // 2) if c["held"] else n
    uni = 4.0 * n * (k + c["halves"] + 1 + (1 if c["groups"] else 0))
    if c["mode"] == "adjoint":
        # the weights and dL/dw read, dL/dmu written; the loadings read, dL/dB written; one
        # product of each of the two factor vectors with the weights and with v per account
        return {"bytes": uni + 8.0 * n * k + 24.0 * m * n, "flops": 4.0 * m * n * k}
    per = 16.0 * n                                    # returns and holdings read, weights written
    per += n / 8.0 if c["excl"] else 0.0
    per += 28.0 * held if c["tax"] else 0.0
    per += 8.0 * n if c["bounds"] else 0.0
    per += 4.0 * n if c["bench"] else 0.0
    per += 8.0 * n if c["mode"] == "warm" else 0.0    # the state read and written
    # one evaluation of the optimality conditions: B^T w and B y
    flops = 4.0 * m * n * (k + c["halves"])
    if c["mode"] == "grad":
        return {"bytes": uni + 8.0 * n * k + m * (per + 16.0 * n), "flops": flops + 4.0 * m * n * k}
    return {"bytes": uni + m * per, "flops": flops}


# ---------------------------------------------------------------------------
# the same problems in 64 bits, without the library: an interior-point method
# on the pieces of every asset's line, then the equality system of the
# pattern it shows
# ---------------------------------------------------------------------------
def _double(t):
    return None if t is None else t.double()


class _Book:
    """The book in float64 with every asset's line cut into the pieces between its bounds and the
    kinks of its trade cost: lengths L, slopes s, side of w0 sg, all [m, n, 5]."""

    def __init__(self, P):
        self.P, m, n = P, P.m, P.n
        dev = P.mu.device
        self.B, self.f, self.d, self.gam = P.B.double(), P.f.double(), P.d.double(), P.gamma.double()
        self.mu, self.w0 = P.mu.double(), P.w0.double()
        el = torch.ones(m, n, dtype=torch.bool, device=dev)
        if P.eligible is not None:
            w = P.eligible.long() & 0xFFFFFFFF
            el = ((w[:, :, None] >> torch.arange(32, device=dev)) & 1).bool().reshape(m, -1)[:, :n]
        lb = P.lb.double()[:, None].expand(m, n) if P.lb_asset is None else P.lb_asset.double()
        ub = P.ub.double()[:, None].expand(m, n) if P.ub_asset is None else P.ub_asset.double()
        zero = torch.zeros((), dtype=torch.float64, device=dev)
        self.lb, ub = torch.where(el, lb, zero), torch.where(el, ub, zero)
        kap = P.kappa.double()[:, None, None]
        cap = torch.isfinite(P.tau)
        b = torch.zeros(m, n, 3, dtype=torch.float64, device=dev)
        t = torch.zeros(m, n, 4, dtype=torch.float64, device=dev)
        if P.tax_ptr is not None:
            acc = torch.repeat_interleave(torch.arange(m, device=dev), P.tax_ptr.diff().long())
            b[acc, P.tax_asset.long()] = P.tax_brk.double()
            t[acc, P.tax_asset.long()] = P.tax_slope.double()
        self.b, self.t = b, t
        w0 = self.w0[:, :, None]
        pts = torch.cat([w0 - b.flip(2), w0], 2).maximum(self.lb[:, :, None]).minimum(ub[:, :, None])
        pts = torch.cat([self.lb[:, :, None], pts, ub[:, :, None]], 2)
        self.pts, self.L = pts, pts.diff(dim=2)
        self.s = torch.cat([-(kap + t.flip(2)), kap.expand(m, n, 1)], 2)
        self.sg = torch.tensor([-1.0, -1.0, -1.0, -1.0, 1.0], dtype=torch.float64, device=dev)
        self.cap, self.tau = cap, P.tau.double()
        self.wb, self.eta = _double(P.wb), _double(P.eta)
        self.lin = self.mu if self.eta is None else self.eta[:, None] * self.mu
        if self.wb is not None:
            self.lin = self.lin + self.gam[:, None] * self.sigma(self.wb)
        rows, lo, hi = [], [], []
        if P.G:
            rows.append(torch.nn.functional.one_hot(P.group.long(), P.G).double())
            lo.append(P.band_lo.double())
            hi.append(P.band_hi.double())
        if P.H:
            rows.append(P.half.double().t())
            lo.append(P.half_lo.double())
            hi.append(P.half_hi.double())
        self.R = torch.cat(rows, 1) if rows else torch.zeros(n, 0, dtype=torch.float64, device=dev)
        self.lo = torch.cat(lo, 1) if lo else torch.zeros(m, 0, dtype=torch.float64, device=dev)
        self.hi = torch.cat(hi, 1) if hi else torch.zeros(m, 0, dtype=torch.float64, device=dev)

    def sigma(self, w):
        return ((w @ self.B) * self.f) @ self.B.t() + w * self.d

    def objective(self, w):
        e = w if self.wb is None else w - self.wb
        mu = self.mu if self.eta is None else self.eta[:, None] * self.mu
        sold = (self.w0 - w).clamp_min(0.0)
        b, t = self.b, self.t
        tax = t[..., 0] * sold
        for j in range(3):
            tax = tax + (t[..., j + 1] - t[..., j]) * (sold - b[..., j]).clamp_min(0.0)
        kap = self.P.kappa.double()
        return (0.5 * self.gam * (e * self.sigma(e)).sum(1) - (mu * w).sum(1)
                + kap * (w - self.w0).abs().sum(1) + tax.sum(1))


def _interior(D):
    """Mehrotra's predictor-corrector over the pieces t in [0, L], the row values r in [lo, hi] and
    the cap's slack; one step length per account.  Returns t, the piece multipliers and
    the row / cap multipliers."""
    m, n, _ = D.L.shape
    dev = D.L.device
    on = D.L > 0
    L = torch.where(on, D.L, torch.ones_like(D.L))
    X = torch.cat([D.B, D.R, torch.ones(n, 1, dtype=torch.float64, device=dev)], 1)
    k, R = D.B.shape[1], D.R.shape[1]
    K = k + R + 1
    gam, gd = D.gam[:, None], D.gam[:, None] * D.d
    flo, fhi = torch.isfinite(D.lo), torch.isfinite(D.hi)
    lo, hi = torch.where(flo, D.lo, D.hi - 1.0), torch.where(fhi, D.hi, D.lo + 1.0)
    c0 = (D.lb - D.w0).abs().sum(1)
    sc = D.lin.abs().amax(1)[:, None]
    t, tu = 0.5 * L, 0.5 * L            # both distances kept: neither loses its digits
    mu0 = 0.1 * sc * D.pts.amax((1, 2))[:, None]      # every pair starts at the same product
    zl = mu0[..., None] / t
    zu = zl.clone()
    r = 0.5 * (lo + hi)
    rl, ru = r - lo, hi - r
    vl, vu = torch.where(flo, mu0 / rl, 0.0), torch.where(fhi, mu0 / ru, 0.0)
    q = torch.where(D.cap, torch.full_like(D.tau, 0.1), 1.0)
    zq = torch.where(D.cap, mu0[:, 0] / q, torch.zeros_like(D.tau))
    y = torch.zeros(m, R + 1, dtype=torch.float64, device=dev)      # rows, budget
    yc = zq.clone()
    tau = torch.where(D.cap, D.tau, torch.zeros_like(D.tau))
    capf = D.cap.double()
    npairs = 2.0 * on.sum((1, 2)) + flo.sum(1) + fhi.sum(1) + D.cap.sum()

    def step(x, dx, mask):
        a = torch.where((dx < 0) & mask, -x / dx, torch.full_like(x, math.inf))
        return a.flatten(1).amin(1) if a[0].numel() else torch.full((m,), math.inf, dtype=torch.float64, device=dev)

    for _ in range(80):
        w = D.lb + torch.where(on, t, 0.0).sum(2)
        gap = (torch.where(on, t * zl + tu * zu, 0.0).sum((1, 2)) + (rl * vl).sum(1)
               + (ru * vu).sum(1) + capf * q * zq)
        mu = gap / npairs
        g = gam * D.sigma(w) - D.lin + y[:, R:] + (y[:, :R] @ D.R.t() if R else 0.0)
        rd = g[..., None] + D.s + (capf * yc)[:, None, None] * D.sg - zl + zu
        rd = torch.where(on, rd, 0.0)
        rr = -y[:, :R] - vl + vu
        pw = torch.cat([w @ D.R - r, w.sum(1, keepdim=True) - 1.0], 1)
        pc = capf * (c0 + (torch.where(on, t, 0.0) * D.sg).sum((1, 2)) + q - tau)
        done = gap <= 1e-14 * sc[:, 0]                    # these accounts stand still from here on
        if bool(done.all()):
            break
        phi = torch.where(on, 1.0 / (zl / t + zu / tu), 0.0)
        Phi, Psi = phi.sum(2), (phi * D.sg).sum(2)
        den = 1.0 + gd * Phi
        al, be = Phi / den, Psi / den
        de = Phi - gd * Psi * Psi / den
        th = vl / rl + vu / ru
        M = torch.empty(m, K + 1, K + 1, dtype=torch.float64, device=dev)
        for a in range(m):
            M[a, :K, :K] = X.t() @ (X * al[a][:, None])
        M[:, :K, K] = M[:, K, :K] = capf[:, None] * (be @ X)
        M[:, K, K] = torch.where(D.cap, de.sum(1) + q / zq.clamp_min(1e-300), torch.ones_like(q))
        dg = torch.zeros(m, K + 1, dtype=torch.float64, device=dev)
        dg[:, :k] = 1.0 / (gam * D.f)
        if R:
            dg[:, k:k + R] = 1.0 / th
        M += torch.diag_embed(dg)
        LU = torch.linalg.lu_factor(M)

        def newton(ct, cu, cl, ch, cq):
            # ct = target of t zl (t zl + ... = ct), cu of tu zu, cl / ch of the rows, cq of the cap
            r1 = torch.where(on, -(rd + zl - zu) + ct / t - cu / tu, 0.0)
            rw = -(rr + vl - vu) + cl / rl - ch / ru
            pr = (phi * r1).sum(2) / den                   # 1^T D^-1 r1
            ps = (phi * D.sg * r1).sum(2) - gd * Psi * pr  # sigma^T D^-1 r1
            rhs = torch.empty(m, K + 1, dtype=torch.float64, device=dev)
            rhs[:, :K] = pr @ X
            rhs[:, k:K] += pw
            if R:
                rhs[:, k:k + R] -= rw / th
            rhs[:, K] = capf * (ps.sum(1) + pc + cq / zq.clamp_min(1e-300) - q)
            x = torch.linalg.lu_solve(*LU, rhs[..., None])[..., 0]
            x = x + torch.linalg.lu_solve(*LU, (rhs - (M @ x[..., None])[..., 0])[..., None])[..., 0]
            u = x[:, :K] @ X.t()
            dyc = capf * x[:, K]
            b = torch.where(on, r1 - u[..., None] - dyc[:, None, None] * D.sg, 0.0)
            dt = phi * b - phi * (gd * (phi * b).sum(2) / den)[..., None]
            dzl, dzu = ct / t - zl - zl / t * dt, cu / tu - zu + zu / tu * dt
            dy = x[:, k:K]
            dr = (rw + dy[:, :R]) / th
            dvl, dvu = cl / rl - vl - vl / rl * dr, ch / ru - vu + vu / ru * dr
            dzq = dyc
            dq = capf * (cq / zq.clamp_min(1e-300) - q - q / zq.clamp_min(1e-300) * dzq)
            return dt, dzl, dzu, dy, dyc, dr, dvl, dvu, dq, dzq

        def length(v):
            dt, dzl, dzu, dy, dyc, dr, dvl, dvu, dq, dzq = v
            c1 = D.cap[:, None]
            pri = torch.stack([step(t, dt, on), step(tu, -dt, on), step(rl, dr, flo),
                               step(ru, -dr, fhi), step(q[:, None], dq[:, None], c1)]).amin(0)
            dua = torch.stack([step(zl, dzl, on), step(zu, dzu, on), step(vl, dvl, flo),
                               step(vu, dvu, fhi), step(zq[:, None], dzq[:, None], c1)]).amin(0)
            return pri, dua

        zt, zr, zc = torch.zeros_like(t), torch.zeros_like(r), torch.zeros_like(q)
        v = newton(zt, zt, zr, zr, zc)
        ap, ad = (x.clamp_max(1.0) for x in length(v))
        a3, d3 = ap[:, None, None], ad[:, None, None]
        g2 = (torch.where(on, (t + a3 * v[0]) * (zl + d3 * v[1]) + (tu - a3 * v[0]) * (zu + d3 * v[2]), 0.0).sum((1, 2))
              + ((rl + ap[:, None] * v[5]) * (vl + ad[:, None] * v[6])).sum(1)
              + ((ru - ap[:, None] * v[5]) * (vu + ad[:, None] * v[7])).sum(1)
              + capf * (q + ap * v[8]) * (zq + ad * v[9]))
        tg = (mu * (g2 / gap).clamp(0.0, 1.0) ** 3).clamp_min(1e-26)
        t3 = tg[:, None, None]
        v = newton(t3 - v[0] * v[1], t3 + v[0] * v[2],
                   torch.where(flo, tg[:, None] - v[5] * v[6], 0.0),
                   torch.where(fhi, tg[:, None] + v[5] * v[7], 0.0), capf * (tg - v[8] * v[9]))
        ap, ad = ((0.9995 * x).clamp_max(1.0) for x in length(v))
        ap = ad = torch.minimum(ap, ad)
        v = [torch.where(done.view(-1, *[1] * (x.dim() - 1)), 0.0, x) for x in v]
        ap, ad = torch.where(done, 0.0, ap), torch.where(done, 0.0, ad)
        a1, d1, a3, d3 = ap[:, None], ad[:, None], ap[:, None, None], ad[:, None, None]
        t, tu = torch.where(on, t + a3 * v[0], t), torch.where(on, tu - a3 * v[0], tu)
        zl, zu = torch.where(on, zl + d3 * v[1], zl), torch.where(on, zu + d3 * v[2], zu)
        y, yc = y + d1 * v[3], yc + ad * v[4]
        r, rl, ru = r + a1 * v[5], rl + a1 * v[5], ru - a1 * v[5]
        vl, vu = vl + d1 * v[6], vu + d1 * v[7]
        q, zq = q + ap * v[8], zq + ad * v[9]
    return t, tu, zl, zu, on, L, y, torch.where(D.cap, yc, torch.zeros_like(yc))


def _optimum(P, c=None):
    """(w, objective, dL/dmu, dL/dB) in float64; the gradients of L = <c, w> where c is given."""
    D = _Book(P)
    t, tu, zl, zu, on, L, y, yc = _interior(D)
    m, n = P.m, P.n
    R = D.R.shape[1]
    # a piece is inside when both distances exceed their multipliers on the account's scale
    sc = D.lin.abs().amax(1)[:, None, None] / D.pts.amax((1, 2))[:, None, None]
    inside = on & (t * sc > zl) & (tu * sc > zu)
    free = inside.any(2)
    full = on & ~inside & (t > tu)
    w = D.lb + torch.where(full, L, 0.0).sum(2)
    piece = torch.where(inside, 1.0, 0.0).argmax(2)
    act = (y[:, :R].abs() > 1e-7 * D.lin.abs().amax(1)[:, None])
    v = torch.zeros_like(w)
    for a in range(m):
        F = torch.nonzero(free[a])[:, 0]
        if not F.numel():
            continue
        gam, BF = D.gam[a], D.B[F]
        w[a, F] = 0.0
        j = piece[a, F]
        rows = [torch.ones(len(F), dtype=torch.float64, device=w.device)]
        h = [1.0 - w[a].sum()]
        for g in torch.nonzero(act[a])[:, 0].tolist():
            rows.append(D.R[F, g])
            h.append((D.hi if y[a, g] > 0 else D.lo)[a, g] - w[a] @ D.R[:, g])
        if bool(D.cap[a]) and float(yc[a]) > 1e-7 * float(D.lin[a].abs().max()):
            rows.append(D.sg[j])
            X = ~free[a]
            h.append(D.tau[a] - (w[a] - D.w0[a])[X].abs().sum() + (D.sg[j] * D.w0[a, F]).sum())
        C, h = torch.stack(rows), torch.stack(h)
        H = gam * ((BF * D.f) @ BF.t() + torch.diag(D.d[F]))
        wx = w[a].clone()
        rhs = D.lin[a, F] - D.s[a, F, j] - gam * ((BF * D.f) @ (D.B.t() @ wx))
        chol = torch.linalg.cholesky(H)
        solve = lambda z: torch.cholesky_solve(z, chol)  # noqa: E731
        HC, Hr = solve(C.t().contiguous()), solve(rhs[:, None])[:, 0]
        S = torch.linalg.pinv(C @ HC, rtol=1e-12, hermitian=True)
        w[a, F] = Hr - HC @ (S @ (C @ Hr - h))
        if c is not None:
            Hc = solve(c[a, F][:, None])[:, 0]
            v[a, F] = Hc - HC @ (S @ (C @ Hc))
    dB = None
    if c is not None:
        e = w if D.wb is None else w - D.wb
        gv, ge = D.gam[:, None] * ((v @ D.B) * D.f), D.gam[:, None] * ((e @ D.B) * D.f)
        dB = -(v.t() @ ge + e.t() @ gv)
        if D.eta is not None:
            v = D.eta[:, None] * v
    return w, D.objective(w), v, dB


def exact(case, seed):
    c = dict(_BASE, **case)
    if c["m"] * c["n"] > 1_000_000:
        return None                                   # minutes, not seconds
    P, g = _inputs(c, seed)
    if c["mode"] in ("grad", "adjoint"):
        w, obj, dmu, dB = _optimum(P, torch.randn(c["m"], c["n"], dtype=torch.float64, device="cuda:0", generator=g))
        if c["mode"] == "adjoint":
            return {"dmu": dmu, "dB": dB}
        return {"w": w, "obj": obj, "status": None, "dmu": dmu, "dB": dB}
    if c["mode"] == "warm":
        P.mu += (1e-4 * torch.randn(P.m, P.n, dtype=torch.float64, device="cuda:0", generator=g)).float()
        w, obj, _, _ = _optimum(P)
        return {"w": w, "obj": obj, "status": None, "state": None}
    w, obj, _, _ = _optimum(P)
    return {"w": w, "obj": obj, "status": None}
