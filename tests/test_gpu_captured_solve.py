"""Solves after replays of captured assemblies.  A replay writes the pattern of
its capture into the context's buffers, whatever the last call had there; a
solve must take the column windows and places of the pattern that is there.
Compared with a context that assembled the same system eagerly: the resident
CG and the three launches give the same bits."""
import numpy as np
import pytest

from gpu_helpers import random_velocity, require_gpu, to_dev
from paper_2008_00409_amd import meshgen as mg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return require_gpu()


@pytest.fixture(scope="module")
def B():
    from paper_2008_00409_amd import binding
    return binding


def solved(ctx, b):
    dv, info = ctx.cloth_pcg_solve(b, tol=1e-8, precond="block")
    return dv.cpu().numpy().tobytes(), info["iters"], info["sweeps"]


def capture(torch, ctx, x, v, dtype):
    b = torch.empty_like(x)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        ctx.cloth_assemble(x, v, dtype, b=b)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        ctx.cloth_assemble(x, v, dtype, b=b)
    torch.cuda.synchronize()
    return graph, b


@pytest.mark.parametrize("dtype", ["f16", "f64"])
@pytest.mark.parametrize("nx,ny", [(23, 19), (60, 50)])
def test_solves_after_replays(torch, B, nx, ny, dtype):
    c, cs = mg.config_contact(nx, ny)
    contacts = (cs.verts, cs.weights, cs.normals, cs.eta, cs.kc)
    x, v = to_dev(torch, c.x0), to_dev(torch, random_velocity(c, 0.02, seed=8))
    want = {}
    for with_contacts in (False, True):
        ctx = B.Context.from_cloth(c)
        try:
            if with_contacts:
                ctx.cloth_set_contacts(*contacts)
            want[with_contacts] = solved(ctx, ctx.cloth_assemble(x, v, dtype))
        finally:
            ctx.close()
    ctx = B.Context.from_cloth(c)
    try:
        def eager(with_contacts):
            ctx.cloth_set_contacts(*contacts) if with_contacts else ctx.cloth_set_contacts()
            return ctx.cloth_assemble(x, v, dtype)

        def replay(with_contacts):
            graph, b = graphs[with_contacts]
            b.zero_()
            graph.replay()
            torch.cuda.synchronize()
            return b

        assert solved(ctx, eager(True)) == want[True]      # the buffers have grown before the first capture
        assert solved(ctx, eager(False)) == want[False]
        graphs = {False: capture(torch, ctx, x, v, dtype)}
        assert solved(ctx, replay(False)) == want[False]
        assert solved(ctx, eager(True)) == want[True]
        assert solved(ctx, replay(False)) == want[False]
        eager(True)
        graphs[True] = capture(torch, ctx, x, v, dtype)
        for last in (False, True, False):
            assert solved(ctx, eager(last)) == want[last]
            eager(last)
            assert solved(ctx, replay(True)) == want[True]
            assert solved(ctx, replay(False)) == want[False]
            assert solved(ctx, replay(True)) == want[True]
    finally:
        ctx.close()
