"""The value pass keeps the element records of a group of four rows in LDS as
long as they fit (704 chunks of 16 bytes: 12 a triangle, 7 or, with the
lookahead force, 9 a hinge) and reads the rest directly.  Closed fans whose
centres are numbered one after the other put four rows of `n` triangles and
`n` hinges each into one group: far below, just below and above the limit, at
a row's own limit (16 triangles and 16 hinges), and in groups with a last row
missing; against the FP64 oracle, at the bars of the other assembly tests."""
import numpy as np
import pytest

from gpu_helpers import random_velocity, require_gpu, to_dev
from paper_2008_00409_amd import meshgen as mg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return require_gpu()


def fans(n, count):
    """`count` closed fans of n triangles, the centres numbered first, one
    centre pinned, one rim vertex pinned."""
    ang = 2 * np.pi * np.arange(n) / n
    rest = np.zeros((count * (n + 1), 3))
    tris = []
    for k in range(count):
        rest[k, 0] = 3.0 * k
        rim = count + k * n + np.arange(n)
        rest[rim, 0] = 3.0 * k + np.cos(ang)
        rest[rim, 1] = np.sin(ang)
        tris += [[k, rim[j], rim[(j + 1) % n]] for j in range(n)]
    pinned = np.zeros(len(rest), np.uint8)
    pinned[[count - 1, count + 1]] = 1
    x0 = rest + 1e-3 * np.random.default_rng(n).uniform(-1, 1, rest.shape)
    x0[pinned == 1] = rest[pinned == 1]
    return mg.Cloth(f"fans-{n}", rest, np.array(tris, dtype=np.int32), np.full(len(rest), 1e-3), pinned, x0,
                    np.zeros_like(rest), 0.01, 1e-8, 1, [(0, len(rest))], [(0, len(tris))])


@pytest.mark.parametrize("rhs_mode", [1, 0])
@pytest.mark.parametrize("n,count", [(3, 1), (4, 4), (8, 4), (9, 4), (10, 4), (12, 7), (16, 4), (16, 5)])
def test_records_in_lds_and_beyond(torch, oracle_mod, n, count, rhs_mode):
    from paper_2008_00409_amd import binding as B
    c = fans(n, count)
    v = random_velocity(c, 0.05, seed=2)
    P = oracle_mod.Problem.from_cloth(c, oracle_mod.Material(rhs_mode=rhs_mode))
    A = P.assemble(c.x0, v)
    ctx = B.Context.from_cloth(c, rhs_mode=rhs_mode)
    try:
        x = to_dev(torch, c.x0)
        diag = torch.empty_like(x)
        b = ctx.cloth_assemble(x, to_dev(torch, v), "f64", diag=diag)
        rowptr, colidx, vals, D = (a.cpu().numpy() for a in ctx.cloth_export_blocks(solver_blocks=False))
        b, diag = b.cpu().numpy(), diag.cpu().numpy()
    finally:
        ctx.close()
    np.testing.assert_array_equal(rowptr, A.rowptr)
    np.testing.assert_array_equal(colidx, A.colidx)
    vals, D = vals.reshape(-1, 3, 3), D.reshape(-1, 3, 3)
    scale = np.repeat(np.array([np.abs(A.vals[A.rowptr[i]:A.rowptr[i + 1]]).max() for i in range(P.nv)]),
                      np.diff(A.rowptr))
    assert (np.abs(vals - A.vals).reshape(-1, 9).max(axis=1) / scale).max() <= 1e-12
    np.testing.assert_allclose(b, A.b, rtol=1e-10, atol=1e-10 * np.abs(A.b).max())
    np.testing.assert_allclose(diag, A.diag, rtol=1e-10)
    np.testing.assert_allclose(D, A.D, rtol=0, atol=1e-12 * np.abs(A.vals).max())
