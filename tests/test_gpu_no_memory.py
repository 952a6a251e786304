"""A solve with contacts when the caller's allocator has no more memory: it needs
none beyond what earlier assemblies and solves took (the resident CG's places,
which it would like, are left out), and gives the same bits."""
import pytest

from gpu_helpers import random_velocity, require_gpu, to_dev
from paper_2008_00409_amd import meshgen as mg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f64", "f16"])
def test_contact_solve_without_memory(dtype):
    torch = require_gpu()
    from paper_2008_00409_amd import binding as B

    class Stingy(B.TorchAllocator):
        empty = False
        refused = 0

        def _alloc(self, nbytes, user):
            if self.empty:
                self.refused += 1
                return None
            return super()._alloc(nbytes, user)

    c, cs = mg.config_contact(23, 19)
    x, v = to_dev(torch, c.x0), to_dev(torch, random_velocity(c, 0.02, seed=8))
    out = []
    for stingy in (False, True):
        allocator = Stingy()
        ctx = B.Context.from_cloth(c, allocator=allocator)
        try:
            ctx.cloth_pcg_solve(ctx.cloth_assemble(x, v, dtype), precond="block")
            ctx.cloth_set_contacts(cs.verts, cs.weights, cs.normals, cs.eta, cs.kc)
            for _ in range(2):
                b = ctx.cloth_assemble(x, v, dtype)
                allocator.empty = stingy
                dv, info = ctx.cloth_pcg_solve(b, tol=1e-8, precond="block")
                out.append((dv.cpu().numpy().tobytes(), info))
                allocator.empty = False
            assert (allocator.refused > 0) == stingy
        finally:
            ctx.close()
    assert all(o == out[0] for o in out)
