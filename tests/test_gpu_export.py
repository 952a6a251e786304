"""The exported blocks at the edges of the export kernel's split (four rows a
workgroup, 16 columns at a time): row counts of every remainder, rows of 2 to 64
columns, rows with and without a stored diagonal block.

The exported matrix must be the one cloth_spmv applies.  Bar: both sides sum at
most 64 x 3 products in FP64, and the true diagonal block is itself such a sum:
1e-13 of the sum of the products' magnitudes."""
import numpy as np
import pytest

from gpu_helpers import random_velocity, require_gpu, sheet, to_dev
from test_gpu_wide_rows import fan_cloth

pytestmark = pytest.mark.gpu

CLOTHS = [("sheet", 2, 2), ("sheet", 5, 1 + 4), ("sheet", 13, 2), ("sheet", 9, 3), ("sheet", 29, 23),
          ("fan", 14, 0), ("fan", 15, 0), ("fan", 16, 0), ("fan", 31, 0), ("fan", 32, 0), ("fan", 47, 0), ("fan", 63, 0)]


@pytest.fixture(scope="module")
def torch():
    return require_gpu()


@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16", "f16"])
@pytest.mark.parametrize("kind,nx,ny", CLOTHS)
def test_export_is_the_applied_matrix(torch, kind, nx, ny, dtype):
    from paper_2008_00409_amd import binding as B
    c = sheet(nx, ny, seed=4, flips=0.1 if nx > 20 else 0.0) if kind == "sheet" else fan_cloth(nx)
    ctx = B.Context.from_cloth(c)
    try:
        ctx.cloth_assemble(to_dev(torch, c.x0), to_dev(torch, random_velocity(c)), dtype)
        z = np.random.default_rng(6).normal(size=c.rest.shape)
        for solver in (False, True):
            rowptr, colidx, vals, D = (a.cpu().numpy() for a in ctx.cloth_export_blocks(solver_blocks=solver))
            rows = np.repeat(np.arange(c.nv), np.diff(rowptr))
            vals = vals.reshape(-1, 3, 3)
            want, size = np.zeros_like(z), np.zeros_like(z)
            np.add.at(want, rows, np.einsum("kab,kb->ka", vals, z[colidx]))
            np.add.at(size, rows, np.einsum("kab,kb->ka", np.abs(vals), np.abs(z[colidx])))
            off = rows != colidx
            sums = np.zeros((c.nv, 3, 3))
            np.add.at(sums, rows[off], np.abs(vals[off]))
            size += np.einsum("iab,ib->ia", sums, np.abs(z))
            got = ctx.cloth_spmv(to_dev(torch, z), solver_blocks=solver).cpu().numpy()
            eps = 1e-13 if not solver or dtype == "f64" else 1e-5   # the solver's product sums in FP32 otherwise
            assert np.all(np.abs(got - want) <= eps * size)
            # the diagonal: m I + D - the row's other blocks
            offs = np.zeros((c.nv, 3, 3))
            np.add.at(offs, rows[off], vals[off])
            diag = D.reshape(-1, 3, 3) + c.mass[:, None, None] * np.eye(3) - offs
            got = np.zeros_like(diag)
            got[rows[~off]] = vals[~off]
            assert np.all(np.abs(got - diag) <= 1e-13 * (sums + c.mass[:, None, None] + np.abs(D.reshape(-1, 3, 3))))
    finally:
        ctx.close()
