"""The network's kernels at the edges of their work split: part of one tile of
16 vertices, whole tiles, an odd tile (the weight gradient takes them in
pairs), and more tiles than one pass of the grid takes (3,072).  The kernels'
own features go through the oracle's network.

Bars.  Each hidden value is rounded to BF16 on both sides, so the two may differ
by one unit in the last place, 2^-7 of the value at most, for each of the three
layers: that bound is carried forward through the absolute weights.  A gradient
passes at most seven such roundings of 2^-8 relative: 7 x 2^-8 < 3e-2 per
tensor."""
import numpy as np
import pytest

from gpu_helpers import random_velocity, require_gpu, sheet, to_dev

pytestmark = pytest.mark.gpu

GRIDS = [(3, 2), (5, 3), (4, 4), (8, 4), (11, 3), (12, 4), (223, 222)]


@pytest.fixture(scope="module")
def torch():
    return require_gpu()


def network(M, seed):
    params = M.init_params(seed)
    rng = np.random.default_rng(seed)
    params[3][0] *= 30.0
    for p in params:
        p[1] = 0.05 * rng.normal(size=p[1].shape)
        p[0], p[1] = M.bf16_round(p[0]), p[1].astype(np.float32).astype(np.float64)
    return params


def setup(torch, nx, ny):
    from oracle import mlp as M
    from paper_2008_00409_amd import binding as B
    c = sheet(nx, ny, seed=5)
    ctx = B.Context.from_cloth(c)
    x, v = to_dev(torch, c.x0), to_dev(torch, random_velocity(c, 0.05, seed=5))
    prev = 0.01 * np.random.default_rng(5).normal(size=c.rest.shape)
    prev[c.pinned == 1] = 0
    prev_d = to_dev(torch, prev)
    diag = torch.empty((c.nv, 3), dtype=torch.float64, device="cuda")
    b = ctx.cloth_assemble(x, v, "f32", diag=diag)
    params = network(M, 5)
    ctx.ws_set_params(M.flatten(params))
    F = ctx.ws_features(x, v, b, prev_d).cpu().numpy().astype(np.uint16)[:c.nv, :27]
    X = (F.astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    edges = [np.linalg.norm(c.rest[c.tris[:, k]] - c.rest[c.tris[:, (k + 1) % 3]], axis=1).mean() for k in range(3)]
    return M, c, ctx, (x, v, b, prev_d), prev, diag.cpu().numpy(), params, X, float(np.mean(edges)) / c.h


@pytest.mark.parametrize("nx,ny", GRIDS)
def test_prediction(torch, nx, ny):
    M, c, ctx, args, prev, diag, params, X, sv = setup(torch, nx, ny)
    try:
        dv0 = ctx.ws_predict(*args).cpu().numpy()
        y, hs = M.forward(params, X, bf16=True)
        err = np.zeros_like(X)
        for k, (W, _) in enumerate(params):
            err = err @ np.abs(W)
            if k < 3:
                err += 2.0 ** -7 * (np.abs(hs[k]) + err)
        err += 2.0 ** -16 * np.abs(y) + 1e-6     # FP32 sums
        free = c.pinned == 0
        assert np.all(np.abs(dv0 - prev - sv * y)[free] <= sv * err[free])
        assert np.all(dv0[~free] == 0)
    finally:
        ctx.close()


@pytest.mark.parametrize("nx,ny", GRIDS)
def test_gradient(torch, nx, ny):
    M, c, ctx, args, prev, diag, params, X, sv = setup(torch, nx, ny)
    try:
        dv0 = ctx.ws_predict(*args)
        Ad = ctx.cloth_spmv(dv0).cpu().numpy()
        got, _ = ctx.ws_gradient(*args)
        y, hs = M.forward(params, X, bf16=True)
        b = args[2].cpu().numpy()
        _, gy = M.energy_loss_grad(lambda z: Ad, b, diag, dv0.cpu().numpy(), c.pinned, sv)
        want = M.flatten(M.backward(params, X, hs, gy, bf16=True))
        o = 0
        for rows, cols in M.SHAPES:
            for n in (rows * cols, cols):
                rel = np.linalg.norm(got[o:o + n] - want[o:o + n]) / np.linalg.norm(want[o:o + n])
                assert rel < 3e-2, (o, n, rel)
                o += n
    finally:
        ctx.close()
