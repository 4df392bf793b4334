"""Recursive update with groups of 64 points on both sides of the grouped
gather's limit (512 distinct rows of P) in one batch, and batches at the edges
of the weight kernel (16 columns, 64 row lanes, 1024 rows in flight).

Against the batch ridge solution with the bound of the update's tests (1e-9),
and the batched plan against the update bit for bit."""
import numpy as np
import pytest
import torch

import oracle as O
from helpers import dev, host
from paper_2509_26222_amd import api, synth

pytestmark = pytest.mark.gpu
TOL = 1e-9


def patch(ctx, p, grid, xy, z, batch):
    N = grid.N
    return dict(grid=grid, w=torch.zeros(N, dtype=torch.float64, device="cuda"),
                P=torch.eye(N, dtype=torch.float64, device="cuda") * (p.R / p.lam),
                xy=dev(xy), z=dev(z), batch=batch, pose=(np.eye(3), np.zeros(3)),
                pts=dev(np.zeros((1, 3)), torch.float32),
                f=torch.empty(1, dtype=torch.float32, device="cuda"),
                grad=torch.empty((1, 2), dtype=torch.float32, device="cuda"),
                resid=torch.empty(1, dtype=torch.float32, device="cuda"),
                jac=torch.empty((1, 6), dtype=torch.float32, device="cuda"))


@pytest.mark.parametrize("nx,ny,m,batch", [
    (36, 37, 320, 320), (36, 37, 300, 128), (8, 8, 257, 256), (13, 5, 90, 17), (9, 7, 40, 15),
    (3, 1, 33, 16), (20, 20, 600, 513), (16, 1, 1100, 1025)])
@pytest.mark.parametrize("scattered", [False, True])
def test_update_and_plan(ctx, nx, ny, m, batch, scattered):
    p = api.Params()
    rng = np.random.default_rng(nx * m + batch)
    c = synth.grid_centers(rng, nx, ny, 0.5, jitter=0.1)
    grid = ctx.grid(p, dev(c))
    xy = rng.uniform(0.0, [0.5 * nx, 0.5 * ny], size=(m, 2))
    xy[: m // 3] *= 0.15          # a third of the points touch few centers
    if not scattered:
        xy = xy[np.lexsort((xy[:, 0], np.floor(xy[:, 1] / 1.5)))]
    z = np.sin(xy[:, 0]) + 0.02 * rng.normal(size=m)
    a = patch(ctx, p, grid, xy, z, batch)
    ctx.update(p, grid, a["w"], a["P"], a["xy"], a["z"], batch=batch)
    wb, Pb = O.ridge_batch(xy, z, c, p.sigma, p.cutoff, 0.0, p.lam, p.R)
    assert np.linalg.norm(host(a["w"]) - wb) <= TOL * np.linalg.norm(wb)
    assert np.abs(host(a["P"]) - Pb).max() <= TOL * np.abs(Pb).max()
    b = patch(ctx, p, grid, xy, z, batch)
    plan = api.Batched(ctx, p, [b], dim=3, eval_prec="f32", gemm_prec="f64")
    plan.run()
    assert plan.sync() == -1
    assert torch.equal(a["w"], b["w"]) and torch.equal(a["P"], b["P"])
    plan.close()
