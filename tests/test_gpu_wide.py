"""GPU tests of the fused iteration pass of wide books (few accounts, no
turnover cap, float32 contractions, n >= 8,192): every sum keeps the order of
the four passes, so the ADMM state after a block equals theirs bit for bit
(settings.profile runs the four passes); and of the null directions swept by
row blocks (n >= 16,384 or so) against the oracle."""
import numpy as np
import pytest

from workloads import make_config
from _gpu_helpers import run_gpu, check_account

pytestmark = pytest.mark.gpu

SHAPES = [
    # name, overrides, settings: chunk edges, every compiled width, account counts
    ("c5", dict(N=8192, M=1, k=100, held=(200, 300)), {}),                      # 160 columns
    ("c5", dict(N=8193, M=3, k=100, held=(200, 300)), {}),
    ("c5", dict(N=8320, M=16, k=70, groups=40, held=(200, 300)), {}),           # 128
    ("c5", dict(N=20001, M=2, k=128, groups=40, held=(200, 300)), {}),          # 192
    ("c5", dict(N=10001, M=2, k=80, groups=0, band_halfwidth=None, held=(200, 300)),
     dict(precision=0)),                                                        # 96
    ("c5", dict(N=8300, M=2, k=100, groups=20, held=(200, 300), halfspaces=5, asset_bounds=True,
                benchmark=True, elig=(0.5, 1.0)), {}),
    ("c5", dict(N=9000, M=2, k=100, held=None, tax=False), {}),                 # dense holdings
]


@pytest.mark.parametrize("name,over,settings", SHAPES)
def test_state_equals_the_four_passes(name, over, settings):
    from paper_2606_23367_amd.solver import Solver, to_device
    uni, book = make_config(name, 41, **over)
    P = to_device(uni, book)
    print(f"case {name} {over}", flush=True)
    states = []
    for profile in (0, 1):
        s = Solver(0)
        out = s.solve(P, rho=10.0, max_iter=40, check_every=20, want_state=True, profile=profile,
                      **settings)
        states.append((out["state"].cpu().numpy(), out["iters"].cpu().numpy(), s.stats()))
    assert states[1][2]["iter_kernel_ms"] > 0.0
    assert np.array_equal(states[0][1], states[1][1])
    assert np.array_equal(states[0][0], states[1][0])


@pytest.mark.parametrize("hw", [1e-3, 5e-3])
def test_null_directions_by_row_blocks(hw):
    uni, book = make_config("c5", 42, N=17000, M=2, k=30, groups=20, band_halfwidth=hw,
                            held=(300, 300), ub=2e-3)
    print(f"case bands {hw}", flush=True)
    host, _ = run_gpu(uni, book, rho=10.0)
    for a in range(book.m):
        check_account(uni, book, a, host)
