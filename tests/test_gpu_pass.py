"""GPU tests of the certification pass that one workgroup runs per account
(n <= 5,120): the order of its phases, seen where most of its 16 waves have no
rows and run ahead of the first."""
import numpy as np
import pytest

from oracle.kkt import residuals
from oracle.problem import account, n_rows
from workloads import make_config
from _gpu_helpers import check_account, check_reported_diagnostics

pytestmark = pytest.mark.gpu


def _solve(uni, book, repeats=1, **settings):
    import torch
    from paper_2606_23367_amd.solver import Solver, to_device
    P, s, runs = to_device(uni, book), Solver(0), []
    for _ in range(repeats):
        out = s.solve(P, **settings)
        torch.cuda.synchronize()
        runs.append({k: v.cpu().numpy() for k, v in out.items()})
    return runs, s.stats()


def _check_diagnostics(uni, book, host):
    for a in range(book.m):
        P = account(uni, book, a)
        r = residuals(P, host["w"][a], host["nu"][a], host["lam_band"][a] if n_rows(P) else None,
                      host["lam_cap"][a])
        check_reported_diagnostics(host, a, r)


# 256 accounts whose free rows pin every multiplier (no null direction, so no
# sweep with its barriers between the gradient scale and the diagnostics): the
# first wave reads the scale's partials while the others store the diagnostics'
@pytest.mark.parametrize("n", [20, 40, 200])
def test_gradient_scale_survives_the_diagnostics(n):
    print(f"case n {n}", flush=True)
    uni, book = make_config("c1", 51, N=n, M=256, k=5, ub=0.2)
    runs, _ = _solve(uni, book, repeats=12, rho=0.05)
    assert np.all(runs[0]["status"] == 0)
    for other in runs[1:]:
        for key in ("w", "obj", "r_prim", "r_dual", "r_comp", "status"):
            assert np.array_equal(runs[0][key], other[key]), key
    _check_diagnostics(uni, book, runs[0])


# free sets too large for the first passes (no trade cost, loose boxes): the gate
# sends the accounts back to the iterations until their pattern repeats, so
# every gated pass hands its bookkeeping to the next one
def test_gated_accounts_resume():
    print("case gated", flush=True)
    uni, book = make_config("c2", 52, N=600, M=24, k=8, groups=3, kappa=0.0, gamma=1000.0, ub=0.05)
    runs, st = _solve(uni, book, repeats=4, rho=1.0, check_every=20, max_iter=4000)
    assert st["polish_gated"] > 0 and st["iterations"] > 20
    assert np.all(runs[0]["status"] == 0)
    for other in runs[1:]:
        for key in ("w", "obj", "r_dual", "iters"):
            assert np.array_equal(runs[0][key], other[key]), key
    _check_diagnostics(uni, book, runs[0])


# optima at a vertex of the box (64 names at ub = 1 / 64, the rest at 0): no free
# row, so every system over the free rows is empty; by one workgroup and by the
# row blocks, and the gradient there (the weights do not move: zero)
@pytest.mark.parametrize("n,m", [(64, 3), (200, 8), (6000, 2)])
def test_patterns_without_free_rows(n, m):
    import torch
    from paper_2606_23367_amd.solver import Solver, to_device
    print(f"case vertex n {n}", flush=True)
    uni, book = make_config("c1", 53, N=n, M=m, k=3, ub=1.0 / 64, w0="zero")
    # 64 names clear of the rest (returns stay float32 values)
    book.mu[:, :64] = (book.mu[:, :64] + 0.25).astype(np.float32)
    book.eligible[:, 200:] = False
    s = Solver(0)
    out = s.solve(to_device(uni, book), rho=10.0)
    host = {k: v.cpu().numpy() for k, v in out.items()}
    assert np.all(host["status"] == 0)
    _check_diagnostics(uni, book, host)
    # (an account may end one pattern short, a free row held at its bound by the budget)
    want = np.where(np.arange(n) < 64, 1.0 / 64, 0.0)
    at = [a for a in range(m) if np.array_equal(host["w"][a], want)]
    assert at, "no account ends without free rows"
    for a in range(min(m, 3)):
        check_account(uni, book, a, host)
    g = torch.ones((m, n), dtype=torch.float64, device="cuda:0")
    dmu, dB = s.adjoint(g)
    assert np.all(dmu.cpu().numpy()[at] == 0.0)
    assert np.all(np.isfinite(dB.cpu().numpy()))
