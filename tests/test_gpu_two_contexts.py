"""Contexts are independent: two threads solve on their own contexts and streams
at once, one with wide windows and one with narrow ones (their resident launches
each take the whole chip and different amounts of LDS), and each solve gives the
bits of the same solve alone."""
import threading

import pytest

from gpu_helpers import random_velocity, require_gpu, sheet, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,precond", [("f64", "block"), ("f16", "block"), ("f32", "jacobi")])
def test_two_threads(dtype, precond):
    torch = require_gpu()
    from paper_2008_00409_amd import binding as B
    jobs = []
    for c in (sheet(363, 363, seed=31, bumps=False, delaunay=False), sheet(363, 180, seed=33, bumps=False, delaunay=False)):
        ctx = B.Context.from_cloth(c)
        b = ctx.cloth_assemble(to_dev(torch, c.x0), to_dev(torch, random_velocity(c, 0.05, seed=2)), dtype)
        want = ctx.cloth_pcg_solve(b, tol=1e-9, maxit=60, precond=precond, raise_on_error=False)
        jobs.append((ctx, b, want, torch.cuda.Stream()))
    torch.cuda.synchronize()
    failures = []

    def solve(ctx, b, want, stream):
        try:
            with torch.cuda.stream(stream):
                dv = torch.empty_like(b)
                for k in range(25):
                    dv.zero_()
                    _, info = ctx.cloth_pcg_solve(b, dv=dv, tol=1e-9, maxit=60, precond=precond, raise_on_error=False)
                    stream.synchronize()
                    if info != want[1] or not torch.equal(dv, want[0]):
                        failures.append((k, info, want[1]))
        except Exception as e:      # reported by the test's own thread
            failures.append(e)

    threads = [threading.Thread(target=solve, args=j) for j in jobs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for ctx, *_ in jobs:
        ctx.close()
    assert not failures, failures[:3]
