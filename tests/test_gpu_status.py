"""The status word around the mesh's pattern: a context whose mesh has a row past
the limits reports it with its assemblies, not before the first; every later
assembly on the held pattern reports it again, also after one that was not
finite."""
import pytest

from gpu_helpers import random_velocity, require_gpu, to_dev
from test_gpu_wide_rows import fan_cloth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return require_gpu()


@pytest.fixture(scope="module")
def B():
    from paper_2008_00409_amd import binding
    return binding


@pytest.mark.parametrize("n", [63, 64, 300])   # the last that fits, 65 columns, 600 corners
def test_nothing_is_reported_before_the_first_assembly(torch, B, n):
    c = fan_cloth(n)
    x, v = to_dev(torch, c.x0), to_dev(torch, random_velocity(c))
    ctx = B.Context.from_cloth(c)
    try:
        for instances in (None, [0, c.nv]):
            if instances is not None:
                ctx.set_instances(instances)
            ctx.check()
            with pytest.raises(B.PclothError, match="PC_ERR_ARG.*nothing assembled"):
                ctx.cloth_pcg_solve(torch.zeros_like(x))
        ctx.cloth_assemble(x, v, "f64")
        if n <= 63:
            ctx.check()
        else:
            with pytest.raises(B.PclothError, match="PC_ERR_CAPACITY"):
                ctx.check()
    finally:
        ctx.close()


def test_row_limits_stay_with_the_held_pattern(torch, B):
    c = fan_cloth(64)
    x, v = to_dev(torch, c.x0), to_dev(torch, random_velocity(c))
    bad = v.clone()
    bad[3, 1] = float("nan")
    ctx = B.Context.from_cloth(c)
    try:
        for u in (v, v, bad, v, bad, bad, v):
            b = ctx.cloth_assemble(x, u, "f32")
            for _ in range(2):
                with pytest.raises(B.PclothError, match="PC_ERR_CAPACITY"):
                    ctx.check()
            with pytest.raises(B.PclothError, match="PC_ERR_CAPACITY"):
                ctx.cloth_pcg_solve(b, maxit=50)
    finally:
        ctx.close()
