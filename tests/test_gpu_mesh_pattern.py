"""The mesh's pattern, laid out once, against a context made for the one
assembly: after other storage types, states, schedules and instances, with rows
past the row groups' incidences and past the limits, and in a captured graph.
The same kernels run on the same values: the same bits."""
import numpy as np
import pytest

from gpu_helpers import random_velocity, require_gpu, sheet, to_dev
from paper_2008_00409_amd import meshgen as mg
from test_gpu_wide_rows import fan_cloth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return require_gpu()


@pytest.fixture(scope="module")
def B():
    from paper_2008_00409_amd import binding
    return binding


def exported(ctx, b, diag):
    out = (b, diag, *ctx.pattern(), *ctx.cloth_export_blocks(True, True), *ctx.cloth_export_blocks(True, False))
    return [a.cpu().numpy().tobytes() for a in out]


def assembled(torch, ctx, x, v, dtype):
    diag = torch.empty_like(x)
    return exported(ctx, ctx.cloth_assemble(x, v, dtype, diag=diag), diag)


def fresh(torch, B, c, x, v, dtype, instances=None):
    ctx = B.Context.from_cloth(c)
    try:
        if instances is not None:
            ctx.set_instances(instances)
        return assembled(torch, ctx, x, v, dtype)
    finally:
        ctx.close()


@pytest.mark.parametrize("make", [lambda: sheet(2, 2), lambda: sheet(13, 5, seed=4), lambda: sheet(29, 23, seed=3),
                                  lambda: fan_cloth(16), lambda: fan_cloth(17), lambda: fan_cloth(63)])
def test_assemblies_on_the_held_pattern(torch, B, make):
    c = make()
    ctx = B.Context.from_cloth(c)
    try:
        for seed, dtype, scale in ((1, "f16", 1.0), (2, "f16", 1e-3), (3, "f64", 1.0), (4, "bf16", 1.0), (5, "f32", 1.0),
                                   (6, "f16", 1.0)):
            x = to_dev(torch, c.x0 + scale * 1e-4 * np.random.default_rng(seed).normal(size=c.x0.shape))
            v = to_dev(torch, random_velocity(c, 0.05, seed=seed))
            if seed == 4:
                ctx.set_option(B.PC_OPT_SPMV_SLICES_PER_BLOCK, 4)
            assert assembled(torch, ctx, x, v, dtype) == fresh(torch, B, c, x, v, dtype)
    finally:
        ctx.close()


def test_instances(torch, B):
    c = mg.config_batch(seed=91, sizes=[13, 40, 9, 27, 2, 3])
    bounds = [r[0] for r in c.sheet_ranges] + [c.nv]
    x, v = to_dev(torch, c.x0), to_dev(torch, random_velocity(c, 0.05, seed=2))
    ctx = B.Context.from_cloth(c)
    try:
        for instances in (None, bounds, [0, c.nv], bounds):
            if instances is not None:
                ctx.set_instances(instances)
            for dtype in ("f16", "f32"):
                assert assembled(torch, ctx, x, v, dtype) == fresh(torch, B, c, x, v, dtype, instances)
    finally:
        ctx.close()


def test_rows_past_the_limits_are_reported_each_time(torch, B):
    c = fan_cloth(64)   # 65 block columns at the centre
    x, v = to_dev(torch, c.x0), to_dev(torch, random_velocity(c))
    ctx = B.Context.from_cloth(c)
    try:
        for _ in range(3):
            b = ctx.cloth_assemble(x, v, "f64")
            with pytest.raises(B.PclothError, match="PC_ERR_CAPACITY"):
                ctx.cloth_pcg_solve(b)
    finally:
        ctx.close()


def test_captured_assembly(torch, B):
    c = sheet(29, 23, seed=3, flips=0.1)
    x, v = to_dev(torch, c.x0), to_dev(torch, random_velocity(c, 0.05, seed=2))
    x2 = to_dev(torch, c.x0 + 1e-4 * np.random.default_rng(7).normal(size=c.x0.shape))
    ctx = B.Context.from_cloth(c)
    try:
        want = [assembled(torch, ctx, y, v, "f16") for y in (x, x2)]
        xs, b, diag = x.clone(), torch.empty_like(x), torch.empty_like(x)
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            ctx.cloth_assemble(xs, v, "f16", b=b, diag=diag)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            ctx.cloth_assemble(xs, v, "f16", b=b, diag=diag)
        for k in (0, 1, 1, 0):
            assert assembled(torch, ctx, (x2, x)[k], v, "f16") == want[1 - k]
            xs.copy_((x, x2)[k])
            b.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert exported(ctx, b, diag) == want[k]
    finally:
        ctx.close()
