"""Support counts taken in LDS, on both sides of their rules: the largest mesh
that fits and one node more, the largest reach and one more, one and several
workgroups' shares of points, points off a 16-byte boundary. The nodes
accepted are those of the oracle, exactly."""
import numpy as np
import pytest
import torch

import oracle as O
from helpers import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,r,n", [
    (1, 1, 0.5, 9000), (192, 192, 0.5, 511), (192, 192, 0.5, 512), (36865, 1, 0.6, 8192),
    (20, 13, 7.5, 8200), (20, 13, 7.6, 8200), (64, 16, 0.0, 5000), (101, 99, 1.2, 12289),
    (40, 30, 0.5, 0), (40, 30, 0.5, 1)])
@pytest.mark.parametrize("shift", [0, 1])
def test_counts(ctx, nx, ny, r, n, shift):
    rng = np.random.default_rng(nx + n)
    xy = rng.uniform([-4.5, -4.5], [0.5 * nx + 4.5, 0.5 * ny + 4.5], size=(n, 2))
    xy[: n // 4] = [0.25 * nx, 0.25 * ny]  # many on one spot
    if n > 100:
        xy[50:56] = [[np.nan, 1.0], [1.0, np.inf], [-np.inf, 1.0], [1e300, 1.0], [0.25, 0.75],
                     [0.25 + r, 0.25]]
    buf = torch.zeros(2 * n + 1, dtype=torch.float64, device="cuda")
    q = buf[shift:shift + 2 * n].view(n, 2)
    q.copy_(torch.from_numpy(xy))
    roi = (0.0, 0.0, 0.5 * nx, 0.5 * ny)
    with np.errstate(invalid="ignore", over="ignore"):
        for thr in (0, 2):
            got = host(ctx.select_centers(q, roi, 0.5, r, thr, O.RADIUS))
            assert np.array_equal(got, O.select_centers(xy, roi, 0.5, r, thr, O.RADIUS))


@pytest.mark.parametrize("nx,ny,r", [(40, 33, 5.5), (40, 33, 5.6), (25, 24, 7.4),
                                     (26, 25, 7.4), (16, 16, 7.4)])
@pytest.mark.parametrize("n", [30, 511, 1025, 2047, 2048])
def test_counts_of_few_points(ctx, nx, ny, r, n):
    """Reach 12 to 16 cells, with meshes on both sides of the nodes that a
    point may test where there are few of them."""
    rng = np.random.default_rng(n)
    xy = rng.uniform([-4.5, -4.5], [0.5 * nx + 4.5, 0.5 * ny + 4.5], size=(n, 2))
    roi = (0.0, 0.0, 0.5 * nx, 0.5 * ny)
    for thr in (0, n // 3):
        got = host(ctx.select_centers(dev(xy), roi, 0.5, r, thr, O.RADIUS))
        assert np.array_equal(got, O.select_centers(xy, roi, 0.5, r, thr, O.RADIUS))
