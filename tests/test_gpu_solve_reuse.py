"""What a context keeps between solves must not show: solves on one context,
through changes of block type, contacts, schedule and start, give the bits of
a fresh context's; dv may be b itself; a refused matrix leaves dv alone."""
import numpy as np
import pytest

from gpu_helpers import random_velocity, require_gpu, sheet, to_dev
from paper_2008_00409_amd import meshgen as mg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return require_gpu()


@pytest.fixture(scope="module")
def B():
    from paper_2008_00409_amd import binding
    return binding


def solve(torch, B, ctx, c, v, dtype, precond, contacts, spb, warm):
    ctx.set_option(B.PC_OPT_SPMV_SLICES_PER_BLOCK, spb)
    ctx.cloth_set_contacts(*contacts) if contacts is not None else ctx.cloth_set_contacts()
    b = ctx.cloth_assemble(to_dev(torch, c.x0), to_dev(torch, v), dtype)
    dv = to_dev(torch, 1e-3 * v)
    dv, info = ctx.cloth_pcg_solve(b, dv=dv, tol=1e-6, precond=precond, warm=warm)
    return dv.cpu().numpy(), info


def test_one_context_through_changes(torch, B):
    c, cs = mg.config_contact(23, 19)
    v = random_velocity(c, 0.05, seed=3)
    contacts = (cs.verts, cs.weights, cs.normals, cs.eta, cs.kc)
    steps = [("f16", "block", None, 8, 0), ("f64", "jacobi", None, 8, 0), ("f16", "jacobi", contacts, 8, 1),
             ("f32", "block", contacts, 4, 0), ("bf16", "block", None, 8, 1), ("f16", "block", None, 4, 0),
             ("f16", "block", None, 8, 0), ("f64", "block", contacts, 8, 1)]
    ctx = B.Context.from_cloth(c)
    try:
        for step in steps:
            d1, i1 = solve(torch, B, ctx, c, v, *step)
            fresh = B.Context.from_cloth(c)
            try:
                d0, i0 = solve(torch, B, fresh, c, v, *step)
            finally:
                fresh.close()
            assert i1 == i0, step
            assert np.array_equal(d1.view(np.uint64), d0.view(np.uint64)), step
    finally:
        ctx.close()


@pytest.mark.parametrize("dtype", ["f16", "f64"])
@pytest.mark.parametrize("window", [0, 1])
def test_dv_may_be_b(torch, B, dtype, window):
    c = sheet(33, 31, seed=5)
    v = random_velocity(c, 0.05, seed=4)
    ctx = B.Context.from_cloth(c)
    try:
        ctx.set_option(B.PC_OPT_LDS_WINDOW, window)
        b = ctx.cloth_assemble(to_dev(torch, c.x0), to_dev(torch, v), dtype)
        d0, i0 = ctx.cloth_pcg_solve(b, tol=1e-9)
        d1, i1 = ctx.cloth_pcg_solve(b, dv=b, tol=1e-9)
        assert i1 == i0 and torch.equal(d1, d0)
    finally:
        ctx.close()


@pytest.mark.parametrize("dtype", ["f16", "f64"])
def test_a_refused_matrix_leaves_dv_alone(torch, B, dtype):
    c = sheet(33, 31, seed=5)
    ctx = B.Context.from_cloth(c)
    try:
        x, v = to_dev(torch, c.x0), to_dev(torch, random_velocity(c, 0.05, seed=4))
        v[500, 1] = float("nan")
        b = ctx.cloth_assemble(x, v, dtype)
        dv = torch.full_like(x, 7.0)
        with pytest.raises(B.PclothError, match="PC_ERR_NONFINITE.*right-hand side"):
            ctx.cloth_pcg_solve(b, dv=dv)
        assert bool((dv == 7.0).all())
        v[500, 1] = 0.0
        b = ctx.cloth_assemble(x, v, dtype)        # the context works on
        dv, info = ctx.cloth_pcg_solve(b, dv=dv, tol=1e-6)
        assert info["rel_res_true"] <= 1e-6
    finally:
        ctx.close()
