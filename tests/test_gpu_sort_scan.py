"""Sorting points by their bins and the prefix sums under it, at the edges of
their chunks (256 or 1024 items) and tiles (8192 counts): the permutation is numpy's
stable argsort of the bins, and the sums (through the row pointers of the Gram
pattern and the accepted nodes of a selection) are exact."""
import numpy as np
import pytest
import torch

import oracle as O
from helpers import dev, host
from paper_2509_26222_amd import api, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 2, 5, 63, 64, 255, 256, 257, 1025, 16_385, 200_001])
@pytest.mark.parametrize("n", [3, 40, 130])  # up to 130 x 130: 45 x 45 bins and more
def test_sort_is_stable(ctx, n, m):
    p = api.Params()
    rng = np.random.default_rng(n + m)
    c = synth.grid_centers(rng, n, n, 0.5, jitter=0.0)
    grid = ctx.grid(p, dev(c))
    xy = rng.uniform(-1.0, 0.5 * n + 1.0, size=(m, 2))
    xy[m // 2:] = xy[m // 2]  # half of the points in one bin
    xo, zo, perm = ctx.sort_points(grid, dev(xy), dev(np.arange(m, dtype=np.float64)))
    pm = host(perm)
    assert np.array_equal(np.sort(pm), np.arange(m))
    assert np.array_equal(host(xo), xy[pm]) and np.array_equal(host(zo), pm.astype(np.float64))
    # equal points keep their order, whatever their bin
    same = pm[np.all(xy[pm] == xy[m // 2], axis=1)]
    assert np.array_equal(same, np.sort(same))
    # the bins of a bin-sorted sequence are contiguous: each (x, y) cell once
    h = p.cutoff * np.sqrt(p.sigma ** 2 + p.sigma_eps ** 2) * (1.0 + 1e-3)  # the bins' side
    x0, y0 = c.min(0) - h
    bins = (np.clip(np.floor((xy[pm, 1] - y0) / h), 0, grid.nby - 1) * grid.nbx +
            np.clip(np.floor((xy[pm, 0] - x0) / h), 0, grid.nbx - 1))
    off = np.abs((xy[pm] - [x0, y0]) / h - np.rint((xy[pm] - [x0, y0]) / h)).min(1) > 1e-9
    assert np.all(np.diff(bins[off]) >= 0)
    order = np.flatnonzero(np.diff(bins) == 0)
    assert np.all(pm[order] < pm[order + 1])


@pytest.mark.parametrize("m", [49_151, 49_152, 49_153, 131_073])
@pytest.mark.parametrize("n", [3, 20, 100])
def test_sort_on_both_sides_of_the_chunk_rule(ctx, n, m):
    p = api.Params()
    rng = np.random.default_rng(m)
    grid = ctx.grid(p, dev(synth.grid_centers(rng, n, n, 0.5, jitter=0.0)))
    xy = rng.uniform(0.0, 0.5 * n, size=(m, 2))
    xo, _, perm = ctx.sort_points(grid, dev(xy))
    pm = host(perm)
    assert np.array_equal(np.sort(pm), np.arange(m)) and np.array_equal(host(xo), xy[pm])
    # sorting the sorted points changes nothing, and ties keep their order
    assert np.array_equal(host(ctx.sort_points(grid, xo)[2]), np.arange(m))
    h = p.cutoff * p.sigma * (1.0 + 1e-3)
    q = (xy[pm] - (0.25 - h)) / h  # bins of the grid; points on an edge left out
    cell = np.clip(np.floor(q), 0, [grid.nbx - 1, grid.nby - 1])
    key = cell[:, 1] * grid.nbx + cell[:, 0]
    ok = np.abs(q - np.rint(q)).min(1) > 1e-9
    assert np.all(np.diff(key[ok]) >= 0)
    assert np.all(np.diff(pm[ok])[np.diff(key[ok]) == 0] > 0)


@pytest.mark.parametrize("n", [1, 63, 1024, 8191, 8192, 8193, 16_385, 40_000])
def test_prefix_sums(ctx, n):
    xy = np.stack([0.5 * np.arange(n) + 0.25, np.full(n, 0.25)], 1)
    keep = np.random.default_rng(n).random(n) < 0.6
    keep[-1] = True
    roi = (0.0, 0.0, 0.5 * n, 0.5)
    got = host(ctx.select_centers(dev(xy[keep]), roi, 0.5, 0.1, 0, O.RADIUS))
    assert np.array_equal(got, O.candidate_mesh(roi, 0.5)[0][keep])
    # lines of at most 13,000 centers, out of each other's reach
    per = min(n, 13_000)
    j = np.arange(n) % per
    last = np.where(np.arange(n) // per == (n - 1) // per, (n - 1) % per, per - 1)
    grid = ctx.grid(api.Params(), dev(np.stack([0.5 * j, 20.0 * (np.arange(n) // per)], 1)))
    rowptr, colidx = ctx.gram_pattern(api.Params(), grid)
    r = int(np.floor(2 * 3.0 * 0.5 / 0.5 + 1e-9))
    assert np.array_equal(np.diff(host(rowptr)), np.minimum(j + r, last) - np.maximum(j - r, 0) + 1)
    assert int(rowptr[-1]) == colidx.shape[0]
