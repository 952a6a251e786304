"""Resident launches that give up waiting.  PC_OPT_RESIDENT_POLLS bounds every
wait from the host: with 0 each workgroup leaves at its first meeting, with a
few polls some leave there, some later, and some finish.  Every kernel ends
normally, and the solve restarts from what the iterate holds with three launches
per iteration and still meets its tolerance, measured here with the FP64 blocks'
product."""
import numpy as np
import pytest

from gpu_helpers import random_velocity, require_gpu, sheet, to_dev
from paper_2008_00409_amd import meshgen as mg

pytestmark = pytest.mark.gpu

TOL = 1e-7


@pytest.fixture(scope="module")
def torch():
    return require_gpu()


@pytest.fixture(scope="module")
def B():
    from paper_2008_00409_amd import binding
    return binding


def system(torch, B, c, dtype, instances=None, contacts=None):
    ctx = B.Context.from_cloth(c)
    if instances is not None:
        ctx.set_instances(instances)
    if contacts is not None:
        ctx.cloth_set_contacts(*contacts)
    return ctx, ctx.cloth_assemble(to_dev(torch, c.x0), to_dev(torch, random_velocity(c, 0.05, seed=2)), dtype)


def residual(ctx, b, dv, bounds):
    """Largest ||b - A dv|| / ||b|| of an instance, A with its FP64 blocks."""
    r = b - ctx.cloth_spmv(dv)
    return max(float(r[i:j].norm() / b[i:j].norm()) for i, j in zip(bounds, bounds[1:]))


@pytest.mark.parametrize("dtype,precond", [("f16", "block"), ("bf16", "jacobi"), ("f32", "block"), ("f64", "jacobi")])
@pytest.mark.parametrize("shape", ["small", "wide", "batch", "contact"])
def test_solves_whose_launches_give_up(torch, B, shape, dtype, precond):
    instances = contacts = None
    if shape == "small":
        c = sheet(43, 31, seed=5)
    elif shape == "wide":                        # 8 pairs a workgroup
        c = sheet(363, 363, seed=31, bumps=False, delaunay=False)
    elif shape == "batch":
        c = mg.config_batch(seed=91, sizes=[13, 40, 9, 27, 60, 33])
        instances = [r[0] for r in c.sheet_ranges] + [c.nv]
    else:
        c, cs = mg.config_contact(23, 19)
        contacts = (cs.verts, cs.weights, cs.normals, cs.eta, cs.kc)
    bounds = instances or [0, c.nv]
    ctx, b = system(torch, B, c, dtype, instances, contacts)
    try:
        kw = dict(tol=TOL, precond=precond)
        _, want = ctx.cloth_pcg_solve(b, **kw)
        for polls in (0, 1, 3, 10, 30, 100):
            ctx.set_option(B.PC_OPT_RESIDENT_POLLS, polls)
            assert ctx.get_option(B.PC_OPT_RESIDENT_POLLS) == polls
            dv, info = ctx.cloth_pcg_solve(b, **kw)
            # the library's own check is <= TOL; the product here rounds in FP64
            assert residual(ctx, b, dv, bounds) <= TOL * (1 + 1e-6), polls
            assert info["fallback"] == want["fallback"]
            if polls == 0:
                assert ctx.get_option(B.PC_OPT_RESIDENT_OFF) == 64
                assert info["sweeps"] == want["sweeps"]          # the lost one does not count
    finally:
        ctx.close()


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_a_lost_sweep_keeps_its_budget(torch, B, dtype):
    """A refinement sweep that was lost is run again with the iterations it had: the
    budget of later sweeps (three times the longest so far, at least 256) would end
    it early, for a sweep more, or on FP64 blocks where its residual has not halved.
    The first sweep of this sheet at rest takes about 1,600 iterations."""
    c = mg.config_medium()
    ctx = B.Context.from_cloth(c)
    try:
        x = to_dev(torch, c.x0)
        b = ctx.cloth_assemble(x, torch.zeros_like(x), dtype)
        kw = dict(tol=1e-6, precond="block")
        _, want = ctx.cloth_pcg_solve(b, **kw)
        assert want["fallback"] == 0
        ctx.set_option(B.PC_OPT_RESIDENT_POLLS, 0)
        dv, info = ctx.cloth_pcg_solve(b, **kw)
        assert ctx.get_option(B.PC_OPT_RESIDENT_OFF) == 64
        assert info["fallback"] == 0 and info["sweeps"] == want["sweeps"], (info, want)
        assert residual(ctx, b, dv, [0, c.nv]) <= 1e-6 * (1 + 1e-6)
    finally:
        ctx.close()


@pytest.mark.parametrize("dtype,max_sweeps", [("f16", 3), ("f64", 1)])
def test_a_lost_sweep_does_not_count(torch, B, dtype, max_sweeps):
    """The sweeps a caller allows are those that do their work: the iterations of an
    undisturbed solve with the same limit."""
    ctx, b = system(torch, B, sheet(43, 31, seed=5), dtype)
    try:
        kw = dict(tol=1e-9, precond="block", max_sweeps=max_sweeps, maxit=1000, raise_on_error=False)
        _, want = ctx.cloth_pcg_solve(b, **kw)
        ctx.set_option(B.PC_OPT_RESIDENT_POLLS, 0)
        _, info = ctx.cloth_pcg_solve(b, **kw)
        assert ctx.get_option(B.PC_OPT_RESIDENT_OFF) == 64
        assert info["sweeps"] == want["sweeps"] and info["status"] == want["status"], (info, want)
        assert abs(info["iters"] - want["iters"]) <= 2 + 0.02 * want["iters"], (info, want)
    finally:
        ctx.close()


def test_a_loss_is_remembered(torch, B):
    """The solves after a loss run without resident launches until 64 have, then 128
    after the second loss in a row; setting the option lets the next one try again."""
    c = sheet(43, 31, seed=5)
    ctx, b = system(torch, B, c, "f64")
    try:
        def solve():
            assert ctx.cloth_pcg_solve(b, tol=1e-2)[1]["sweeps"] == 1
            return ctx.get_option(B.PC_OPT_RESIDENT_OFF)

        assert solve() == 0
        ctx.set_option(B.PC_OPT_RESIDENT_POLLS, 0)
        for between in (64, 128):
            assert [solve() for _ in range(between + 1)] == list(range(between, -1, -1))
        assert solve() == 256
        ctx.set_option(B.PC_OPT_RESIDENT_POLLS, 0)
        assert ctx.get_option(B.PC_OPT_RESIDENT_OFF) == 0 and solve() == 64 and solve() == 63
        ctx.set_option(B.PC_OPT_RESIDENT_POLLS, 2_000_000)
        assert solve() == 0
        with pytest.raises(B.PclothError, match="PC_ERR_ARG"):
            ctx.set_option(B.PC_OPT_RESIDENT_OFF, 0)
    finally:
        ctx.close()


def test_autotuner_does_not_time_a_loss(torch, B):
    """64 iterations that were not run would be the fastest of all; three launches
    an iteration take more than 3 us."""
    c = sheet(43, 31, seed=5)
    ctx, b = system(torch, B, c, "f64")
    try:
        ctx.set_option(B.PC_OPT_RESIDENT_POLLS, 0)
        assert ctx.autotune(b, iters=64)["ms_per_iter"] > 3e-3
        dv, _ = ctx.cloth_pcg_solve(b, tol=TOL)
        assert residual(ctx, b, dv, [0, c.nv]) <= TOL * (1 + 1e-6)
    finally:
        ctx.close()


def test_option_range(torch, B):
    ctx = B.Context.from_cloth(sheet(5, 4))
    try:
        assert ctx.get_option(B.PC_OPT_RESIDENT_POLLS) == 2_000_000
        for value in (-1, 2_000_001, 1 << 40):
            with pytest.raises(B.PclothError, match="PC_ERR_ARG"):
                ctx.set_option(B.PC_OPT_RESIDENT_POLLS, value)
    finally:
        ctx.close()
