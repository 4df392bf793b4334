"""The covariance product in its tiled forms, on maps that reach each of them:
blocks of 32x32 alone (2025 centers), blocks of 64x32 alone (2311), both in one
launch (2916), sizes and batches that are no multiple of the blocks or of the
loop's rows; and the same under the two-stream schedule, which splits the tiles
by the rows that the next batch reads.

Reference: the dense Kalman step in numpy, to 16 n eps cond(S) (the step is
backward stable); the one-stream schedule, bit for bit."""
import numpy as np
import pytest
import torch

import oracle as O
from helpers import dev, host
from paper_2509_26222_amd import api, synth

pytestmark = pytest.mark.gpu
EPS = np.finfo(np.float64).eps


def lattice(rng, n):
    nx = int(np.ceil(np.sqrt(n)))
    return nx, synth.grid_centers(rng, nx, nx, 0.5, jitter=0.1, first=n)


@pytest.mark.parametrize("n,m", [(2025, 37), (2311, 37), (2311, 161), (2916, 3), (2901, 161)])
def test_one_batch(ctx, n, m):
    p = api.Params(R=1e-2)
    rng = np.random.default_rng(n + m)
    nx, c = lattice(rng, n)
    xy, z = rng.uniform(0.0, 0.5 * nx, size=(m, 2)), rng.normal(0.0, 0.1, m)
    a = rng.normal(size=(n, 3)) * 0.2
    P0, w0 = np.eye(n) * 0.4 + a @ a.T, rng.normal(0.0, 0.1, n)
    grid = ctx.grid(p, dev(c))
    w, P = dev(w0), dev(P0)
    print(f"tiled n {n} m {m}", flush=True)
    assert ctx.update(p, grid, w, P, dev(xy), dev(z), batch=m) == m
    H = O.regressor_dense(xy, c, p.sigma, p.cutoff, 0.0)
    U = P0 @ H.T
    S = H @ U + p.R * np.eye(m)
    G = np.linalg.solve(S, U.T)
    tol = 16 * n * EPS * np.linalg.cond(S)
    Pg = host(P)
    assert np.array_equal(Pg, Pg.T)
    assert np.abs(Pg - (P0 - U @ G)).max() <= tol * np.abs(P0).max()
    w1 = w0 + G.T @ (z - H @ w0)
    assert np.abs(host(w) - w1).max() <= tol * (np.abs(w0).max() + np.abs(z).max()) * 10


@pytest.mark.parametrize("n", [2025, 2311, 2916])
def test_two_streams(ctx, n):
    p = api.Params()
    rng = np.random.default_rng(n)
    nx, c = lattice(rng, n)
    grid = ctx.grid(p, dev(c))
    # sorted points of a part of the map: batches touch some of the row blocks
    xy = rng.uniform([0.0, 0.1 * nx], [0.4 * nx, 0.4 * nx], size=(700, 2))
    xs, zs, _ = ctx.sort_points(grid, dev(xy), dev(rng.normal(0.0, 0.1, 700)))
    got = []
    for streams in (1, 2):
        print(f"streams {streams} n {n}", flush=True)
        w = torch.zeros(n, dtype=torch.float64, device="cuda")
        P = torch.eye(n, dtype=torch.float64, device="cuda") * (p.R / p.lam)
        ctx.set_update_streams(streams)
        try:
            assert ctx.update(p, grid, w, P, xs, zs, batch=90) == 700
        finally:
            ctx.set_update_streams(1)
        got.append((host(w), host(P)))
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
