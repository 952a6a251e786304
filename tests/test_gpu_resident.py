"""The resident CG (a sweep's iterations in one launch) must give the bits of
the three-launch iteration, which PC_OPT_LDS_WINDOW = 0 selects: at the edges
of slices (64 rows), of workgroups (128, 256, 512 and 1,024 rows) and of the
compute units' number of them, for every block and vector type and both
preconditioners; with instances of mixed sizes, one of them left to the three
launches because its columns are scattered; and with a right-hand side that
is not finite."""
import numpy as np
import pytest

from gpu_helpers import random_velocity, require_gpu, sheet, to_dev
from paper_2008_00409_amd import meshgen as mg

pytestmark = pytest.mark.gpu

SIZES = [(2, 2), (8, 8), (13, 5), (16, 8), (43, 3), (64, 16), (41, 25), (64, 32), (97, 75), (256, 128), (331, 99),
         (256, 256), (251, 262), (512, 256), (363, 363), (512, 512), (513, 512)]


@pytest.fixture(scope="module")
def torch():
    return require_gpu()


@pytest.fixture(scope="module")
def B():
    from paper_2008_00409_amd import binding
    return binding


def both(torch, B, c, dtype, precond, maxit, instances=None, spoil=None, contacts=None):
    """(dv, info) with the resident launches and with three launches."""
    ctx = B.Context.from_cloth(c)
    out = []
    try:
        if instances is not None:
            ctx.set_instances(instances)
        if contacts is not None:
            ctx.cloth_set_contacts(*contacts)
        v = to_dev(torch, random_velocity(c, 0.05, seed=2))
        for window in (1, 0):
            ctx.set_option(B.PC_OPT_LDS_WINDOW, window)
            b = ctx.cloth_assemble(to_dev(torch, c.x0), v, dtype)
            if spoil is not None:
                b.view(-1)[spoil[0]] = spoil[1]
            dv, info = ctx.cloth_pcg_solve(b, tol=1e-9, maxit=maxit, precond=precond, raise_on_error=False)
            out.append((dv.cpu().numpy(), info))
    finally:
        ctx.close()
    return out


def check_same(out):
    (d1, i1), (d0, i0) = out
    assert np.all(np.equal(i1["iters"], i0["iters"])) and np.all(np.equal(i1["sweeps"], i0["sweeps"]))
    assert np.array_equal(d1.view(np.uint64), d0.view(np.uint64))


@pytest.mark.parametrize("dtype,precond", [("f16", "block"), ("bf16", "jacobi"), ("f32", "block"), ("f64", "jacobi")])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_resident_gives_the_three_launch_bits(torch, B, nx, ny, dtype, precond):
    c = sheet(nx, ny, seed=31, bumps=False, delaunay=False)
    check_same(both(torch, B, c, dtype, precond, maxit=19))


@pytest.mark.parametrize("dtype,precond", [("f16", "jacobi"), ("bf16", "block"), ("f32", "jacobi"), ("f64", "block")])
def test_resident_instances_of_mixed_sizes(torch, B, dtype, precond):
    parts = [sheet(7, 9, seed=41), sheet(40, 40, seed=42), sheet(100, 90, seed=43, delaunay=False), sheet(64, 33, seed=44)]
    p = parts[2]                                                  # columns over all of its 9,000 rows
    perm = np.random.default_rng(5).permutation(p.nv)
    inv = np.argsort(perm)
    parts[2] = mg.Cloth("scattered", p.rest[inv], perm[p.tris].astype(np.int32), p.mass[inv], p.pinned[inv],
                        p.x0[inv], p.v0[inv], p.h, p.tol, 1, [(0, p.nv)], [(0, p.nt)])
    begins = np.concatenate([[0], np.cumsum([q.nv for q in parts])]).tolist()
    cat = lambda k: np.concatenate([getattr(q, k) for q in parts])
    tris = np.concatenate([q.tris + begins[i] for i, q in enumerate(parts)]).astype(np.int32)
    c = mg.Cloth("mixed", cat("rest"), tris, cat("mass"), cat("pinned"), cat("x0"), cat("v0"), p.h, p.tol, 1,
                 [(0, begins[-1])], [(0, len(tris))])
    check_same(both(torch, B, c, dtype, precond, maxit=150, instances=begins))


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_resident_reports_a_right_hand_side_that_is_not_finite(torch, B, value):
    c = sheet(40, 30, seed=45)
    (_, i1), (_, i0) = both(torch, B, c, "f16", "block", maxit=40, spoil=(3 * 700, value))
    assert i1["status"] == i0["status"] != 0
    assert i1["iters"] == i0["iters"] and i1["sweeps"] == i0["sweeps"]


@pytest.mark.parametrize("nx,ny", [(5, 4), (23, 19), (90, 70), (150, 130)])
@pytest.mark.parametrize("sheets", [2, 3])
def test_resident_with_contacts_between_sheets(torch, B, sheets, nx, ny):
    """Contacts between neighbouring sheets put columns far below and above a
    workgroup's own rows (up to 2 x 19,500 away): random vertex-face pairs."""
    parts = [sheet(nx, ny, seed=51 + k, bumps=False, delaunay=False) for k in range(sheets)]
    n = nx * ny
    cat = lambda k: np.concatenate([getattr(q, k) for q in parts])
    tris = np.concatenate([q.tris + n * k for k, q in enumerate(parts)]).astype(np.int32)
    x0 = cat("x0")
    for k in range(sheets):
        x0[n * k:n * (k + 1), 2] += 1.5e-3 * k
    c = mg.Cloth("stack", cat("rest"), tris, cat("mass"), cat("pinned"), x0, cat("v0"), 0.01, 1e-6, 1,
                 [(0, sheets * n)], [(0, len(tris))])
    rng = np.random.default_rng(7)
    up = rng.permutation(n)[:max(3, n // 2)]
    low = parts[0].tris[rng.integers(0, len(parts[0].tris), len(up))]
    near = np.array([parts[0].tris[np.argmin(np.abs(parts[0].tris - u).sum(axis=1))] for u in up[:64]])
    low[:len(near)] = near
    verts = np.concatenate([np.column_stack([n * (k + 1) + up, n * k + low]) for k in range(sheets - 1)]).astype(np.int32)
    weights = np.tile([1.0, -0.5, -0.3, -0.2], (len(verts), 1))
    normals = np.tile([0.0, 0.0, 1.0], (len(verts), 1))
    for dtype, precond in (("f16", "block"), ("f32", "jacobi"), ("f64", "block")):
        check_same(both(torch, B, c, dtype, precond, maxit=23, contacts=(verts, weights, normals, 2e-3, 1000.0)))


@pytest.mark.parametrize("count,nx,ny", [(17, 128, 128), (40, 80, 90), (300, 20, 20), (257, 2, 2)])
def test_resident_rounds(torch, B, count, nx, ny):
    """More instances than the chip takes at once: several launches (the last
    shape is one workgroup an instance)."""
    parts = [sheet(nx, ny, seed=61 + k % 3, bumps=False, delaunay=False) for k in range(count)]
    n = nx * ny
    cat = lambda k: np.concatenate([getattr(q, k) for q in parts])
    tris = np.concatenate([q.tris + n * k for k, q in enumerate(parts)]).astype(np.int32)
    c = mg.Cloth("rounds", cat("rest"), tris, cat("mass"), cat("pinned"), cat("x0"), cat("v0"), 0.01, 1e-6, 1,
                 [(0, count * n)], [(0, len(tris))])
    begins = list(range(0, count * n + 1, n))
    for dtype, precond in (("bf16", "block"), ("f32", "block"), ("f64", "jacobi")):
        check_same(both(torch, B, c, dtype, precond, maxit=60, instances=begins))
