"""GPU parity of the factor-space solve of the four passes at every compiled
width, with as many row tiles as a thread sums in one short batch and one more
(settings.profile times the launches of the four passes and so runs them)."""
import pytest

from workloads import make_config
from _gpu_helpers import run_gpu, check_account

pytestmark = pytest.mark.gpu

# factors -> padded columns 32, 64, 96, 128, 160, 192: 512 / columns threads a
# column, four partials each, 128 rows a partial
WIDTHS = [(20, 8192), (50, 4096), (90, 2560), (110, 2048), (120, 1536), (125, 1024)]


@pytest.mark.parametrize("k,rows", WIDTHS)
@pytest.mark.parametrize("more", [0, 1])
def test_row_tiles_of_a_batch(k, rows, more):
    n, groups = rows + more, {120: 20, 125: 40}.get(k, 0)
    print(f"case k {k} groups {groups} n {n}", flush=True)
    uni, book = make_config("c2", 71, N=n, M=1, k=k, ub=max(0.02, 8.0 / n), groups=groups,
                            band_halfwidth=0.02 if groups else None)
    host, st = run_gpu(uni, book, rho=1.0, profile=1)
    assert st["iter_kernel_ms"] > 0.0                        # the four passes ran
    check_account(uni, book, 0, host)
