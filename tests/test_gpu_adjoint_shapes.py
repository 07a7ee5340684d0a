"""GPU adjoint at the edges of its tiles: rows and factors around multiples of
16, account counts around 4 and 16, free sets from a handful to hundreds,
factor counts around the 64 lanes; against the oracle's gradient."""
import numpy as np
import pytest

import oracle
from oracle.adjoint import gradients
from oracle.problem import account
from workloads import make_config
from test_gpu_adjoint import _gpu_adjoint

pytestmark = pytest.mark.gpu

SHAPES = [
    # (n, m, k, groups, gamma)
    (33, 1, 1, 0, 1.0), (48, 3, 15, 3, 1000.0), (95, 4, 16, 4, 1000.0), (130, 5, 17, 4, 100.0),
    (500, 17, 33, 10, 1000.0), (400, 2, 64, 5, 1000.0), (401, 3, 65, 5, 1000.0),
    (600, 2, 128, 20, 1000.0),
]


@pytest.mark.parametrize("n,m,k,groups,gamma", SHAPES)
def test_gradients(n, m, k, groups, gamma):
    uni, book = make_config("c4", 5, N=n, M=m, k=k, gamma=gamma, groups=groups, ub=0.2,
                            band_halfwidth=0.05 if groups else None)
    print(f"case {n} {m} {k} {groups}", flush=True)
    C = np.random.default_rng(5).normal(size=(m, n))
    host, dmu, dB = _gpu_adjoint(uni, book, C, rho=1.0, eps_prim=1e-9, eps_dual=1e-9,
                                 eps_comp=1e-9)
    assert np.all(host["status"] == 0)
    ref, sB = np.zeros_like(dB), 0.0
    for a in range(m):
        P = account(uni, book, a)
        orc = oracle.solve_account(P)
        g_mu, g_B = gradients(P, orc["w"], orc["lam_band"], orc["lam_cap"], C[a])
        scale = max(np.abs(g_mu).max(), np.abs(C[a]).max() / (gamma * uni.d.max()))
        assert np.max(np.abs(dmu[a] - g_mu)) <= 1e-6 * scale, a
        ref += g_B
        # (an all-zero reference is an LP-like vertex: dL/dB = -(v y^T + ...) with v on
        # the scale above)
        sB += scale * np.abs(gamma * uni.f * (uni.B.T @ orc["w"])).max()
    assert np.max(np.abs(dB - ref)) <= 1e-6 * max(np.abs(ref).max(), sB)
