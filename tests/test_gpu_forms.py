"""Which form a block of iterations takes, and that every form ran where the
rule says so: a fresh handle's workspace holds the account-resident blocks'
or the wide pass's copy of B~ only when that form is taken, so its bytes against
a profiled call's (always the four passes) tell the forms apart."""
import numpy as np
import pytest

from workloads import make_config
from _gpu_helpers import check_account

pytestmark = pytest.mark.gpu


def _bytes(P, profile, **settings):
    from paper_2606_23367_amd.solver import Solver
    s = Solver(0)
    out = s.solve(P, profile=profile, **settings)
    return s.stats()["workspace_bytes"], {k: v.cpu().numpy() for k, v in out.items()}


def _form(P, **settings):
    """bytes the call's form takes beyond the four passes, and its outputs"""
    more, out = _bytes(P, 0, **settings)
    four, _ = _bytes(P, 1, **dict(settings, max_iter=1))
    return more - four, out


def _resident_bytes(n, m, quarters, lots):
    tiles = -(-n // 64)
    own = 16 * tiles * quarters * 64 + 16 * m * 64 * tiles + (4 * m * 64 * tiles if lots else 0)
    return own - (16 + 16 + (4 if lots else 0))              # one entry each where not taken


# name, overrides, settings, quarters of the compiled width
RESIDENT = [
    ("c2", dict(N=700, M=3, k=20), dict(rho=1.0), 8),
    ("c3", dict(N=700, M=3, k=95), dict(rho=5.0), 24),
    ("c3", dict(N=513, M=3, k=8, ub=0.02, held=(8, 60)), dict(rho=5.0), 6),
    ("e7", dict(M=300, N=130, k=6, ub=0.05), dict(rho=1.0, alpha=1.8), 6),
    # thousands of accounts on few names (the passes' workgroups cost more)
    ("e7", dict(M=4096, N=64, k=6, ub=0.1), dict(rho=1.0, alpha=1.8), 6),
]


@pytest.mark.parametrize("name,over,settings,quarters", RESIDENT)
def test_account_resident_blocks(name, over, settings, quarters):
    from paper_2606_23367_amd.solver import to_device
    print(f"case {name} {over}", flush=True)
    uni, book = make_config(name, 81, **over)
    P = to_device(uni, book)
    more, host = _form(P, **settings)
    assert more == _resident_bytes(uni.n, book.m, quarters, P.tax_ptr is not None)
    for a in (0, book.m - 1):
        check_account(uni, book, a, host)


@pytest.mark.parametrize("N,k,groups,columns", [(8192, 100, 50, 100), (9001, 70, 0, 72)])
def test_wide_pass(N, k, groups, columns):
    from paper_2606_23367_amd.solver import to_device
    print(f"case wide {N} {k}", flush=True)
    uni, book = make_config("c5", 82, N=N, M=2, k=k, groups=groups,
                            band_halfwidth=0.02 if groups else None, held=(200, 300))
    more, _ = _form(to_device(uni, book), rho=10.0, precision=0, max_iter=50)
    assert more == 4 * 128 * (-(-N // 128)) * columns - 4


# past the line: few held names make the four passes cheap on large books, a cap
# makes a block search its rows (with lots on every name more so)
FOUR = [
    ("c2", dict(N=8192, M=384, k=55, groups=0, band_halfwidth=None, w0="zero"), {}),
    ("c3", dict(N=6000, M=4, k=80), {}),
    ("c3", dict(N=2048, M=512, k=5, ub=0.02, held=(2048, 2048)), {}),
    ("c2", dict(N=700, M=2, k=96, groups=0, band_halfwidth=None), {}),
]


@pytest.mark.parametrize("name,over,settings", FOUR)
def test_four_passes(name, over, settings):
    from paper_2606_23367_amd.solver import to_device
    print(f"case four {name} {over}", flush=True)
    uni, book = make_config(name, 83, **over)
    more, _ = _form(to_device(uni, book), rho=5.0, max_iter=50, **settings)
    assert more == 0


# accounts with and without a cap, of several risk aversions (a factor-space
# block each), with and without lots, in one book of account-resident blocks
@pytest.mark.parametrize("n", [300, 1100])
def test_mixed_accounts(n):
    from paper_2606_23367_amd.solver import to_device
    print(f"case mixed {n}", flush=True)
    uni, book = make_config("c3", 84, N=n, M=9, k=12, ub=0.03, groups=5, band_halfwidth=0.1,
                            held=(10, 60))
    book.tau[::2] = np.inf
    book.gamma[:] = np.resize([1.0, 100.0, 1000.0], 9)
    book.kappa[:] = np.float32(1e-3) * (np.arange(9) % 2)
    P = to_device(uni, book)
    more, host = _form(P, rho=5.0)
    assert more == _resident_bytes(n, 9, 6, True)
    for a in range(9):
        check_account(uni, book, a, host)
