"""GPU tests of the active-set refinement at the edges of its solves: the
constraint system in one wave's lanes and above them, panels of the
factorisation, free sets on either side of the row-space solve, the rows of a
pass by one workgroup."""
import numpy as np
import pytest

from workloads import make_config
from _gpu_helpers import run_gpu, check_account

pytestmark = pytest.mark.gpu

CASES = [
    # narrow bands bind nearly all of them: 1 + groups constraint columns
    # against the 44 one wave solves; factor counts around the panels of 8
    # and the 64 lanes
    dict(N=700, M=3, k=7, groups=42, band_halfwidth=1e-5, ub=0.02),
    dict(N=700, M=3, k=8, groups=43, band_halfwidth=1e-5, ub=0.02),
    dict(N=700, M=3, k=9, groups=44, band_halfwidth=1e-5, ub=0.02),
    dict(N=900, M=2, k=65, groups=64, band_halfwidth=1e-5, ub=0.02),
    dict(N=900, M=2, k=100, groups=63, band_halfwidth=1e-5, ub=0.02),
    # no trade cost and loose boxes: hundreds of free rows (factor space);
    # factor counts at the panel and stride edges
    dict(N=600, M=2, k=16, groups=5, tax=False, kappa=0.0,
         gamma=1000.0, ub=0.05),
    dict(N=600, M=2, k=64, groups=5, tax=False, kappa=0.0,
         gamma=1000.0, ub=0.05),
    dict(N=600, M=2, k=101, groups=5, tax=False, kappa=0.0,
         gamma=1000.0, ub=0.05),
    dict(N=600, M=2, k=127, groups=0, band_halfwidth=None, tax=False, kappa=0.0,
         gamma=1000.0, ub=0.05),
]

# the rows of one workgroup's pass: a handful, around its blocks of 512 and its
# 1,024 threads, the largest it takes and the first it leaves to the row blocks
SIZES = [
    ("c2", dict(N=3, M=2, k=1, groups=0, band_halfwidth=None, ub=0.6)),
    ("c2", dict(N=65, M=2, k=3, groups=4, ub=0.2)),
    ("c5", dict(N=511, M=2, k=30, groups=7, band_halfwidth=1e-3, ub=0.03, held=(60, 90))),
    ("c5", dict(N=1025, M=2, k=33, groups=7, band_halfwidth=1e-3, ub=0.02, held=(60, 90),
                halfspaces=5, asset_bounds=True, benchmark=True, elig=(0.5, 1.0))),
    ("c3", dict(N=2049, M=2, k=20, ub=0.02)),
    ("c5", dict(N=5120, M=2, k=40, groups=10, band_halfwidth=1e-3, ub=0.01, held=(100, 200))),
    ("c5", dict(N=5121, M=2, k=40, groups=10, band_halfwidth=1e-3, ub=0.01, held=(100, 200))),
]


@pytest.mark.parametrize("over", CASES)
def test_against_the_oracle(over):
    uni, book = make_config("c5", 43, held=(60, 90), **over)
    print(f"case {over}", flush=True)
    host, _ = run_gpu(uni, book, rho=10.0, max_iter=4000)
    # (the accounts the oracle itself solves to 1e-11 and the iteration settles
    # within max_iter)
    for a in (1,) if over["groups"] == 44 else (0, 1):
        check_account(uni, book, a, host)


@pytest.mark.parametrize("name,over", SIZES)
def test_rows_of_a_pass(name, over):
    uni, book = make_config(name, 44, **over)
    print(f"case {name} {over}", flush=True)
    host, _ = run_gpu(uni, book, rho=10.0, max_iter=4000)
    for a in range(2):
        check_account(uni, book, a, host)


# a factor of no variance: the book is the one without its column (free sets in
# row space, in factor space, and the row blocks), and so are its gradients
DEAD_FACTOR = [("c2", dict(N=500, M=2, k=9, groups=4, ub=0.05), 1.0),
               ("c5", dict(N=600, M=2, k=40, groups=5, tax=False, kappa=0.0, gamma=1000.0, ub=0.05,
                           held=(60, 90)), 10.0),
               ("c5", dict(N=6000, M=2, k=70, groups=5, tax=False, kappa=0.0, gamma=1000.0, ub=0.05,
                           held=(60, 90)), 10.0)]


@pytest.mark.parametrize("name,over,rho", DEAD_FACTOR)
def test_factor_without_variance(name, over, rho):
    import oracle
    from dataclasses import replace
    from oracle.adjoint import gradients
    from oracle.problem import account
    from test_gpu_adjoint import _gpu_adjoint
    print(f"case dead factor {over}", flush=True)
    uni, book = make_config(name, 45, **over)
    dead = over["k"] // 2
    keep = np.arange(uni.k) != dead
    uni.f[dead] = 0.0
    short = replace(uni, B=np.ascontiguousarray(uni.B[:, keep]), f=uni.f[keep])
    C = np.random.default_rng(45).normal(size=(book.m, uni.n))
    host, dmu, dB = _gpu_adjoint(uni, book, C, rho=rho, eps_prim=1e-9, eps_dual=1e-9, eps_comp=1e-9)
    assert np.all(dB[:, dead] == 0.0)
    ref, bound = np.zeros((uni.n, uni.k - 1)), 0.0
    for a in range(book.m):
        check_account(short, book, a, host)
        P = account(short, book, a)
        orc = oracle.solve_account(P)
        g_mu, g_B = gradients(P, orc["w"], orc["lam_band"], orc["lam_cap"], C[a])
        # (the scale of the other gradient tests: a vertex has a zero gradient)
        scale = max(np.abs(g_mu).max(), np.abs(C[a]).max() / (P.gamma * short.d.max()))
        assert np.max(np.abs(dmu[a] - g_mu)) <= 1e-6 * scale, a
        ref += g_B
        bound += scale * np.abs(P.gamma * short.f * (short.B.T @ orc["w"])).max()
    assert np.max(np.abs(dB[:, keep] - ref)) <= 1e-6 * max(np.abs(ref).max(), bound)
