"""GPU parity of the account-resident iteration blocks (one workgroup runs a
whole block of ADMM iterations of its account) at the edges of their layout:
64-row tiles, one to three tiles a wave, factor widths on both sides of every
compiled width, constraint rows, lots, per-asset bounds and the turnover cap.
Small books take these blocks; settings.profile times the launches of the
four passes and therefore runs them instead, so both paths are compared on
the same books."""
import numpy as np
import pytest

from workloads import make_config
from _gpu_helpers import run_gpu, check_account

pytestmark = pytest.mark.gpu


def _both(uni, book, **settings):
    host, _ = run_gpu(uni, book, **settings)
    four, st = run_gpu(uni, book, profile=1, **settings)
    assert st["iter_kernel_ms"] > 0.0                        # the four passes ran
    for a in range(book.m):
        check_account(uni, book, a, host)
        check_account(uni, book, a, four)


@pytest.mark.parametrize("n", [37, 64, 65, 511, 512, 513, 1024, 1025])
@pytest.mark.parametrize("cap", [False, True])
def test_row_tiles(n, cap):
    print(f"case n {n} cap {cap}", flush=True)
    if cap:
        uni, book = make_config("c3", 31, N=n, M=3, k=8, ub=max(0.01, 8.0 / n),
                                held=(min(8, n // 4), min(60, n // 2)))
        _both(uni, book, rho=5.0)
    else:
        uni, book = make_config("c2", 31, N=n, M=3, k=8, ub=max(0.05, 8.0 / n), groups=0,
                                band_halfwidth=None)
        _both(uni, book, rho=1.0)


# used columns k + 1 (+ 10 bands): 24 / 25, 32 / 33, 44 / 45, 56 / 57, 72 / 73, 84 / 85, 96 / 97
@pytest.mark.parametrize("k", [23, 24, 31, 32, 43, 44, 55, 56, 71, 72, 83, 84, 95, 96])
def test_factor_widths(k):
    print(f"case k {k}", flush=True)
    uni, book = make_config("c3", 32, N=700, M=2, k=k)
    _both(uni, book, rho=5.0)
    uni, book = make_config("c2", 32, N=700, M=2, k=max(k - 10, 1))
    _both(uni, book, rho=1.0)


def test_every_rule_family():
    print("case bands, halfspaces, per-asset bounds, benchmark, lots, masks, cap", flush=True)
    uni, book = make_config("c3", 33, N=1100, M=4, k=20, groups=6, band_halfwidth=0.05,
                            halfspaces=4, half_halfwidth=1e-2, asset_bounds=True, benchmark=True,
                            ub=0.02, cap_slack=0.3)
    _both(uni, book, rho=5.0)


def test_more_accounts_than_compute_units():
    uni, book = make_config("e7", 34, M=300, N=130, k=6, ub=0.05)
    print("case 300 accounts", flush=True)
    host, _ = run_gpu(uni, book, rho=1.0, alpha=1.8)
    four, _ = run_gpu(uni, book, rho=1.0, alpha=1.8, profile=1)
    assert np.all(host["status"] == 0) and np.all(four["status"] == 0)
    for a in (0, 255, 256, 299):
        check_account(uni, book, a, host)
    assert np.max(np.abs(host["w"] - four["w"])) <= 1e-7


def test_state_after_one_block_matches_the_four_passes():
    # the ADMM state itself (v, constraint rows, cap multiplier) after 10
    # iterations: float32 sums in another order (and bf16 splits, 2^-16 a
    # product, in the four passes), scaled by the largest entry
    from paper_2606_23367_amd.solver import Solver, to_device
    for name, over in (("c3", dict(N=900, M=3, k=12)), ("c2", dict(N=900, M=3, k=12))):
        uni, book = make_config(name, 35, **over)
        P = to_device(uni, book)
        print(f"case state {name}", flush=True)
        out = [Solver(0).solve(P, rho=5.0, max_iter=10, check_every=10, want_state=True,
                               profile=pr, precision=0)["state"].cpu().numpy() for pr in (0, 1)]
        mn = book.m * uni.n
        v0, v1 = out[0][:mn], out[1][:mn]
        assert np.max(np.abs(v0 - v1)) <= 1e-4 * np.max(np.abs(v1))
        np.testing.assert_allclose(out[0][mn:], out[1][mn:], rtol=1e-3, atol=1e-6)
