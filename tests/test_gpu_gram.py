"""The information matrix by dense blocks of the points' bins, on both sides
of its rules: up to 128 and up to 256 candidates per bin (one and several
passes over a bin's blocks), more than that (the row-wise kernel), more bins
than one strip holds, fewer points than three for four centers, more bins than
centers, bins without points, points off the grid, a non-finite
height.

Tolerance: an entry is a sum of n_p positive products of two regressor values,
n_p the points in both supports (<= the points of the case). A value's
exponent, at most cutoff^2 / 2 <= 5, has a relative error of 4 eps here and in
the reference, so the value 40 eps, with the exponential and the scale 44; a
product 90, the sum (n_p + 90) eps. Two runs are equal bit for bit."""
import numpy as np
import pytest
import torch

import oracle as O
from helpers import dev, host
from paper_2509_26222_amd import api, synth

pytestmark = pytest.mark.gpu
EPS = np.finfo(np.float64).eps


def assemble(ctx, p, grid, xy, z, **kw):
    rp, ci = ctx.gram_pattern(p, grid)
    vals, b = ctx.assemble_gram(p, grid, dev(xy), dev(z), rp, ci, **kw)
    return host(rp), host(ci), host(vals), host(b)


def check(ctx, p, c, xy, z):
    grid = ctx.grid(p, dev(c))
    print(f"centers {c.shape[0]} points {xy.shape[0]} candidates {grid.max_candidates} "
          f"bins {grid.nbx} x {grid.nby}", flush=True)
    rp, ci, vals, b = assemble(ctx, p, grid, xy, z)
    H, b0 = O.gram(xy, z, c, p.sigma, p.cutoff, p.sigma_eps, p.lam, sparse=True)
    rows = np.repeat(np.arange(c.shape[0]), np.diff(rp))
    ref = np.asarray(H[rows, np.array(ci)]).ravel()
    tol = (xy.shape[0] + 90) * EPS
    assert np.all(np.abs(vals - ref) <= tol * np.abs(ref) + 1e-300)
    ab = O.gram(xy, np.abs(z), c, p.sigma, p.cutoff, p.sigma_eps, p.lam, sparse=True)[1]
    assert np.all(np.abs(b - b0) <= tol * ab + 1e-300)
    again = assemble(ctx, p, grid, xy, z)
    assert np.array_equal(vals, again[2]) and np.array_equal(b, again[3])
    return grid


@pytest.mark.parametrize("res,n,m,lo,hi", [
    (0.5, 17, 500, 1, 128), (0.42, 19, 900, 97, 160), (0.32, 23, 700, 161, 256),
    (0.25, 20, 300, 257, 100_000)])
def test_candidate_counts(ctx, res, n, m, lo, hi):
    p = api.Params()
    rng = np.random.default_rng(n)
    c = synth.grid_centers(rng, n, n - 2, res, jitter=0.2 * res)
    xy = rng.uniform(-2.0, n * res + 2.0, size=(m, 2))
    grid = check(ctx, p, c, xy, rng.normal(size=m))
    assert lo <= grid.max_candidates <= hi


@pytest.mark.parametrize("m", [0, 1, 20249, 20250])
def test_strips_and_empty_bins(ctx, m):
    p = api.Params()
    rng = np.random.default_rng(m)
    c = synth.grid_centers(rng, 180, 150, 0.5, jitter=0.0)
    xy = rng.uniform([-5.0, -5.0], [40.0, 80.0], size=(m, 2))  # the rest has no points
    xy[:1] = 1e4
    grid = check(ctx, p, c, xy, rng.normal(size=m))
    ld = (grid.max_candidates + 15) // 16 * 16
    assert grid.nbx * grid.nby * 8 * ld * ld > 128 << 20


def test_scattered_centers(ctx):
    """More bins than centers: the row-wise kernel, however many the points."""
    rng = np.random.default_rng(11)
    c = np.concatenate([rng.uniform(0.0, 6.0, size=(60, 2)), [[3000.0, 2000.0]]])
    xy = rng.uniform(0.0, 6.0, size=(500, 2))
    grid = check(ctx, api.Params(), c, xy, rng.normal(size=500))
    assert grid.nbx * grid.nby > c.shape[0]


def test_accumulates_and_non_finite_height(ctx):
    p = api.Params()
    rng = np.random.default_rng(3)
    c = synth.grid_centers(rng, 12, 12, 0.5, jitter=0.1)
    xy = rng.uniform(0.0, 6.0, size=(400, 2))
    z = rng.normal(size=400)
    grid = ctx.grid(p, dev(c))
    rp, ci = ctx.gram_pattern(p, grid)
    v, b = ctx.assemble_gram(p, grid, dev(xy[:150]), dev(z[:150]), rp, ci)
    ctx.assemble_gram(p, grid, dev(xy[150:]), dev(z[150:]), rp, ci, v, b, add_lambda=False)
    v1, b1 = ctx.assemble_gram(p, grid, dev(xy), dev(z), rp, ci)
    assert torch.allclose(v, v1, rtol=490 * EPS, atol=0)
    z[7] = np.nan
    _, _, vn, bn = assemble(ctx, p, grid, xy, z)
    hit = O.regressor_dense(xy[7:8], c, p.sigma, p.cutoff, p.sigma_eps)[0] > 0
    assert np.array_equal(np.isnan(bn), hit)
    assert np.array_equal(vn, host(v1)) and np.array_equal(bn[~hit], host(b1)[~hit])


@pytest.mark.parametrize("nx,ny,res,m", [
    (30, 30, 1.0, 2000), (30, 30, 1.0, 9000), (400, 1, 0.5, 350), (400, 1, 0.5, 12_000),
    (2, 300, 0.5, 700), (2, 300, 0.5, 15_000), (10, 10, 0.5, 99), (10, 10, 0.5, 100),
    (1, 1, 0.5, 900), (2, 2, 0.5, 64)])
def test_both_sides_of_the_estimates(ctx, nx, ny, res, m):
    """Sparse and thin lattices and small ones, with few points (row-wise) and
    with many (by blocks)."""
    rng = np.random.default_rng(m)
    c = synth.grid_centers(rng, nx, ny, res, jitter=0.1 * res)
    xy = rng.uniform(-0.5, [nx * res + 0.5, ny * res + 0.5], size=(m, 2))
    check(ctx, api.Params(), c, xy, rng.normal(size=m))


@pytest.mark.parametrize("nx,ny,res,m", [
    (60, 60, 0.75, 5400), (60, 60, 0.75, 14_400), (90, 40, 0.9, 2736), (90, 40, 0.9, 14_400),
    (64, 64, 0.5, 3112), (2000, 2, 0.5, 3040), (2000, 2, 0.5, 16_000)])
def test_lattices_near_the_estimates_line(ctx, nx, ny, res, m):
    """Lattices on which the two forms take about as long: by rows and by blocks."""
    rng = np.random.default_rng(m)
    c = synth.grid_centers(rng, nx, ny, res, jitter=0.1 * res)
    xy = rng.uniform(-0.5, [nx * res + 0.5, ny * res + 0.5], size=(m, 2))
    check(ctx, api.Params(), c, xy, rng.normal(size=m))
