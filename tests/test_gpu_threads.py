"""GPU test of several host threads, a handle and a stream each, on books whose
kernels take different amounts of LDS: a kernel's limit belongs to the process,
so a thread must not lower it under another's launch.  Every call's weights are
those of the same call made alone."""
import threading

import numpy as np
import pytest

from workloads import make_config

pytestmark = pytest.mark.gpu

# (factors, bands): 10, 35, 36 and 41 KB in the factor-space solve of the four
# passes (more than 96 columns: no account-resident block)
BOOKS = [(100, 20), (100, 56), (104, 56), (100, 63)]


def test_books_of_different_lds_sizes():
    import torch
    from paper_2606_23367_amd.solver import Solver, to_device
    jobs = []
    for q, (k, groups) in enumerate(BOOKS):
        uni, book = make_config("c5", 61 + q, N=900, M=3, k=k, groups=groups, band_halfwidth=0.02,
                                ub=0.02, held=(60, 90))
        jobs.append((to_device(uni, book), Solver(0), torch.cuda.Stream()))
    settings = [dict(rho=10.0, check_every=ce) for ce in (50, 40, 30)]

    def run(q):
        P, s, stream = jobs[q]
        with torch.cuda.stream(stream):
            return [s.solve(P, stream=stream, **kw)["w"] for kw in settings]

    print("case alone", flush=True)
    alone = [run(q) for q in range(len(jobs))]
    torch.cuda.synchronize()
    got, errors = [None] * len(jobs), []

    def loop(q):
        try:
            for _ in range(4):
                got[q] = run(q)
        except Exception as e:          # noqa: BLE001 (reported below)
            errors.append((q, e))

    print("case together", flush=True)
    threads = [threading.Thread(target=loop, args=(q,)) for q in range(len(jobs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
    for q in range(len(jobs)):
        for x, y in zip(alone[q], got[q]):
            assert np.array_equal(x.cpu().numpy(), y.cpu().numpy()), q
