"""The FP64 products of the update (V V^T and L^{-1} U^T, one block per wave
straight from global memory) at the edges of their blocks: sizes around 16,
32, 64 and 128, batches that are no multiple of the loop's rows, sizes on
both sides of the rule for small products, and an L^{-1} operand of more than
2^31 bytes (two buffer resources). Reference: the dense Kalman step in numpy
or the same points in other batches, which agree in exact arithmetic.

Tolerance: the step is backward stable; P and w are off by at most a modest
multiple of n eps cond(S) of what is subtracted (S = H P H^T + R I has
cond(S) <= (|H|^2 |P| + R) / R by the norms used below): 16 n eps cond(S)."""
import numpy as np
import pytest
import torch

import oracle as O
from helpers import dev, host
from paper_2509_26222_amd import api, synth

pytestmark = pytest.mark.gpu
EPS = np.finfo(np.float64).eps


def case(n, m, seed):
    """n centers on a 0.5 m mesh, m points over them, a coupled covariance."""
    rng = np.random.default_rng(seed)
    nx = int(np.ceil(np.sqrt(n)))
    c = synth.grid_centers(rng, nx, nx, 0.5, jitter=0.1, first=n)
    xy = rng.uniform(0.0, 0.5 * nx, size=(m, 2))
    a = rng.normal(size=(n, 3)) * 0.2
    return c, xy, rng.normal(0.0, 0.1, m), np.eye(n) * 0.4 + a @ a.T, rng.normal(0.0, 0.1, n)


@pytest.mark.parametrize("n,m", [(15, 33), (16, 64), (17, 1), (33, 95), (64, 97), (65, 128),
                                 (127, 130), (129, 257), (725, 200), (1030, 161)])
def test_one_batch_block_edges(ctx, n, m):
    p = api.Params(R=1e-2)
    c, xy, z, P0, w0 = case(n, m, n + m)
    grid = ctx.grid(p, dev(c))
    w, P = dev(w0), dev(P0)
    print(f"one batch n {n} m {m}", flush=True)
    assert ctx.update(p, grid, w, P, dev(xy), dev(z), batch=m) == m
    H = O.regressor_dense(xy, c, p.sigma, p.cutoff, 0.0)
    U = P0 @ H.T
    S = H @ U + p.R * np.eye(m)
    G = np.linalg.solve(S, U.T)
    tol = 16 * max(n, m) * EPS * np.linalg.cond(S)
    Pg = host(P)
    assert np.array_equal(Pg, Pg.T)
    assert np.abs(Pg - (P0 - U @ G)).max() <= tol * np.abs(P0).max()
    w1 = w0 + G.T @ (z - H @ w0)
    assert np.abs(host(w) - w1).max() <= tol * (np.abs(w0).max() + np.abs(z).max()) * 10


def test_operand_over_two_gib(ctx):
    """17,000 points in one batch (L^{-1}: 17,024^2 doubles, 2.3 GB) against
    batches of 1024: the same state in exact arithmetic."""
    n, m = 400, 17_000
    p = api.Params()
    c, xy, z, _, _ = case(n, m, 5)
    grid = ctx.grid(p, dev(c))
    xs, zs, _ = ctx.sort_points(grid, dev(xy), dev(z))
    got = []
    for batch in (m, 1024):
        print(f"batch {batch}", flush=True)
        w = torch.zeros(n, dtype=torch.float64, device="cuda")
        P = torch.eye(n, dtype=torch.float64, device="cuda") * (p.R / p.lam)
        assert ctx.update(p, grid, w, P, xs, zs, batch=batch) == m
        got.append((host(w), host(P)))
    # cond(S) <= 28 (R/lam)/R + 1 = 2.8e4 of at most 28 active centers per
    # point and P <= R/lam; several hundred points share them
    tol = 16 * m * EPS * 2.8e4
    assert np.abs(got[0][1] - got[1][1]).max() <= tol * (p.R / p.lam)
    assert np.abs(got[0][0] - got[1][0]).max() <= tol * np.abs(got[1][0]).max()
