"""A matrix that the assembly's status word refuses is reported without iterating
on it: no kernel of an iteration runs (counted with the profiler, which samples
the first), dv is untouched, and the context solves the next good one."""
import pytest

from gpu_helpers import random_velocity, require_gpu, sheet, to_dev
from test_gpu_wide_rows import fan_cloth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return require_gpu()


@pytest.fixture(scope="module")
def B():
    from paper_2008_00409_amd import binding
    return binding


@pytest.mark.parametrize("dtype,method,warm", [("f64", "cg", "zero"), ("f16", "cg", "given"), ("bf16", "cg", "zero"),
                                               ("f32", "chronopoulos-gear", "given")])
@pytest.mark.parametrize("window", [1, 0])
@pytest.mark.parametrize("fault", ["limits", "finite"])
def test_no_iterations(torch, B, fault, window, dtype, method, warm):
    c = fan_cloth(64) if fault == "limits" else sheet(33, 31, seed=5)
    x, v = to_dev(torch, c.x0), to_dev(torch, random_velocity(c, 0.05, seed=4))
    bad = v.clone()
    if fault == "finite":
        bad[7, 1] = float("nan")
    ctx = B.Context.from_cloth(c)
    try:
        ctx.set_option(B.PC_OPT_LDS_WINDOW, window)
        b = ctx.cloth_assemble(x, bad, dtype)
        dv = torch.full_like(x, 7.0)
        ctx.profile(1)
        with pytest.raises(B.PclothError, match="PC_ERR_CAPACITY" if fault == "limits" else "PC_ERR_NONFINITE"):
            ctx.cloth_pcg_solve(torch.ones_like(b), dv=dv, maxit=200, method=method, warm=warm)
        assert "spmv" not in ctx.profile_read()
        ctx.profile(0)
        assert bool((dv == 7.0).all())
        if fault == "finite":
            b = ctx.cloth_assemble(x, v, dtype)
            _, info = ctx.cloth_pcg_solve(b, tol=1e-6, method=method)
            assert info["rel_res_true"] <= 1e-6
    finally:
        ctx.close()
