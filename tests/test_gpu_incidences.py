"""The mesh's incidences are laid out once and an assembly with contacts adds
theirs: contacts switched on, changed and off on one context must give what a
fresh context gives, bit for bit.  The row pointers come from scans of one
launch (up to 1,024 rows), two (up to 4,096 tiles) and three."""
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


def outputs(torch, ctx, c, v, contacts):
    ctx.cloth_set_contacts(*contacts) if contacts is not None else ctx.cloth_set_contacts()
    x = to_dev(torch, c.x0)
    diag = torch.empty_like(x)
    b = ctx.cloth_assemble(x, to_dev(torch, v), "f32", diag=diag)
    return [a.cpu().numpy() for a in (b, diag, *ctx.cloth_export_blocks(), *ctx.cloth_export_blocks(False, True)[2:3])]


def test_contacts_on_and_off(torch, B):
    c, cs = mg.config_contact(23, 19)
    v = random_velocity(c, 0.05, seed=3)
    full = (cs.verts, cs.weights, cs.normals, cs.eta, cs.kc)
    part = (cs.verts[::3], cs.weights[::3], cs.normals[::3], cs.eta, cs.kc)
    ctx = B.Context.from_cloth(c)
    try:
        for contacts in (None, part, full, None, full, part):
            got = outputs(torch, ctx, c, v, contacts)
            fresh = B.Context.from_cloth(c)
            try:
                want = outputs(torch, fresh, c, v, contacts)
            finally:
                fresh.close()
            for g, w in zip(got, want):
                assert g.tobytes() == w.tobytes()
    finally:
        ctx.close()


@pytest.mark.parametrize("nx,ny", [(2, 2), (32, 31), (32, 32), (41, 25), (64, 32), (683, 3), (2051, 2050)])
def test_row_pointers(torch, B, nx, ny):
    """Row pointers and columns of a grid triangulation against the columns
    derived from its triangles on the host."""
    rest, tris = mg.grid(nx, ny, 0.01 * (nx - 1), 0.01 * (ny - 1), 0.0)
    nv = len(rest)
    c = mg.Cloth("grid", rest, tris, np.full(nv, 1e-3), np.zeros(nv, np.uint8), rest, np.zeros_like(rest), 0.01, 1e-6,
                 1, [(0, nv)], [(0, len(tris))])
    ctx = B.Context.from_cloth(c)
    try:
        x = to_dev(torch, c.x0)
        ctx.cloth_assemble(x, torch.zeros_like(x), "f32")
        rowptr, colidx = (a.cpu().numpy() for a in ctx.pattern())
        hinges = ctx.hinges()[0]
    finally:
        ctx.close()
    pairs = [tris[:, [0, 1]], tris[:, [1, 2]], tris[:, [2, 0]], hinges[:, [2, 3]]]
    p = np.concatenate([q.astype(np.int64) for q in pairs])
    key = np.concatenate([p[:, 0] * nv + p[:, 1], p[:, 1] * nv + p[:, 0], np.arange(nv, dtype=np.int64) * (nv + 1)])
    key.sort()
    key = key[np.concatenate([[True], key[1:] != key[:-1]])]
    np.testing.assert_array_equal(rowptr, np.concatenate([[0], np.cumsum(np.bincount(key // nv, minlength=nv))]))
    np.testing.assert_array_equal(colidx, key % nv)
