"""The 64x64 blocks of the Cholesky of S (rotating chain with progress words
in LDS): batches around the 16-column panels and the 64-row blocks against
the dense Kalman step in numpy, and a non-positive pivot in every panel.

Centers 10 m apart, so a point at a center sees that center only and S is
the P of the points' centers plus R, which the test chooses. Tolerance: the
step is backward stable, so P and w are off by at most a modest multiple of
n eps cond(S) of the quantities that are subtracted (n = 130 points,
cond(S) <= 1.1e3 by construction): 64 n eps cond(S) |P|."""
import numpy as np
import pytest
import torch

from helpers import dev, host
from paper_2509_26222_amd import api

pytestmark = pytest.mark.gpu
EPS = np.finfo(np.float64).eps


def far_centers(n):
    i = np.arange(n)
    return np.stack([10.0 * (i % 16), 10.0 * (i // 16)], 1).astype(np.float64)


def spd(n, seed):
    """Covariance with eigenvalues in [1e-3, 1], all coupled."""
    rng = np.random.default_rng(seed)
    q, _ = np.linalg.qr(rng.normal(size=(n, n)))
    p = (q * np.geomspace(1e-3, 1.0, n)) @ q.T
    return 0.5 * (p + p.T)


@pytest.mark.parametrize("m", [1, 15, 16, 17, 48, 63, 64, 65, 112, 128, 130])
def test_one_batch_matches_dense_step(ctx, m):
    n = 130
    p = api.Params(R=1e-3)
    c = far_centers(n)
    P0 = spd(n, m)
    rng = np.random.default_rng(100 + m)
    w0, z = rng.normal(size=n), rng.normal(size=m)
    grid = ctx.grid(p, dev(c))
    w, P = dev(w0), dev(P0)
    print(f"one batch of {m}", flush=True)
    assert ctx.update(p, grid, w, P, dev(c[:m]), dev(z), batch=m) == m
    S = P0[:m, :m] + p.R * np.eye(m)
    G = np.linalg.solve(S, P0[:m])
    tol = 64 * n * EPS * np.linalg.cond(S)
    assert np.abs(host(P) - (P0 - P0[:, :m] @ G)).max() <= tol * np.abs(P0).max()
    w1 = w0 + G.T @ (z - w0[:m])
    assert np.abs(host(w) - w1).max() <= tol * (np.abs(w1).max() + np.abs(z).max())


@pytest.mark.parametrize("bad", [0, 15, 16, 37, 63, 64, 100, 129])
def test_bad_pivot_in_any_panel(ctx, bad):
    n = 130
    p = api.Params(R=1e-3)
    c = far_centers(n)
    P0 = np.eye(n)
    P0[bad, bad] = -1.0  # S[bad, bad] = -1 + R
    grid = ctx.grid(p, dev(c))
    w, P = torch.zeros(n, dtype=torch.float64, device="cuda"), dev(P0)
    with pytest.raises(api.RbfError) as e:
        ctx.update(p, grid, w, P, dev(c), dev(np.ones(n)), batch=n)
    assert e.value.status == 3  # RBF_E_NOT_SPD
    assert np.array_equal(host(P), P0) and np.all(host(w) == 0.0)
