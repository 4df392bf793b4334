"""Binned evaluation of few points, read from the grid's arrays without the
packed table, against the packed form, which a call of more points takes: the
same operations on the same values in the same order, so the outputs are equal
bit for bit."""
import numpy as np
import pytest
import torch

from helpers import dev
from paper_2509_26222_amd import api, synth

pytestmark = pytest.mark.gpu
LIMIT = 65536  # largest call that reads the arrays as they are


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("nx,ny,res,Q", [(1, 1, 0.5, 1), (20, 20, 0.5, 1000), (60, 50, 0.2, 3001),
                                         (99, 101, 0.5, LIMIT)])
def test_raw_equals_packed(ctx, dtype, nx, ny, res, Q):
    p = api.Params()
    rng = np.random.default_rng(nx + Q)
    c = synth.grid_centers(rng, nx, ny, res, jitter=0.2 * res)
    grid = ctx.grid(p, dev(c))
    w = dev(rng.normal(size=c.shape[0]))
    R, t = synth.rot_zyx(0.4, 0.05, -0.02), np.array([0.3, -0.2, 0.6])
    n = LIMIT + 1
    world = np.concatenate([rng.uniform(-2.0, [nx * res + 2.0, ny * res + 2.0], size=(n, 2)),
                            rng.normal(size=(n, 1))], 1)
    xyz = (world - t) @ R
    if Q > 64:
        xyz[20:25, 0] = [np.nan, np.inf, -np.inf, 1e30, -1e9]
    bits = torch.int32 if dtype == torch.float32 else torch.int64
    for pts, pose in ((dev(xyz).to(dtype), (R, t)),
                      (dev(world[:, :2]).to(dtype).contiguous(), None)):
        full = ctx.eval(p, grid, w, pts, pose=pose)
        part = ctx.eval(p, grid, w, pts[:Q], pose=pose)
        for key, v in part.items():
            if v is not None:
                assert torch.equal(v.view(bits), full[key][:Q].view(bits)), key


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("nx,ny", [(1, 1), (2, 1), (3, 3), (7, 5), (20, 20), (45, 31)])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_non_finite_weight_stays_with_its_center(ctx, dtype, nx, ny, bad):
    """A masked slot behind the arrays' end reads no weight: a weight that is
    not finite, the first center's among them, reaches the same points in both
    forms."""
    p = api.Params()
    rng = np.random.default_rng(nx)
    c = synth.grid_centers(rng, nx, ny, 0.5, jitter=0.1)
    grid = ctx.grid(p, dev(c))
    n = LIMIT + 1
    xy = rng.uniform(-1.0, [nx * 0.5 + 1.0, ny * 0.5 + 1.0], size=(n, 2))
    pts = dev(xy).to(dtype)
    bits = torch.int32 if dtype == torch.float32 else torch.int64
    for at in {0, c.shape[0] // 2, c.shape[0] - 1}:
        w = rng.normal(size=c.shape[0])
        w[at] = bad
        full = ctx.eval(p, grid, dev(w), pts)
        part = ctx.eval(p, grid, dev(w), pts[:2001])
        for key in ("f", "grad"):
            a, b = part[key], full[key][:2001]
            assert torch.equal(a.isnan(), b.isnan()), (at, key)
            ok = ~a.isnan()
            assert torch.equal(a[ok].view(bits), b[ok].view(bits)), (at, key)


@pytest.mark.parametrize("dtype,lim", [(torch.float32, 3_800_000), (torch.float64, 7_000_000)])
@pytest.mark.parametrize("nx,res", [(40, 0.15), (60, 0.3), (70, 0.5)])
def test_both_sides_of_the_candidates_rule(ctx, dtype, lim, nx, res):
    """The last call that reads the arrays and the first that packs them, by the
    candidates of the grid."""
    p = api.Params()
    rng = np.random.default_rng(nx)
    grid = ctx.grid(p, dev(synth.grid_centers(rng, nx, nx, res, jitter=0.1 * res)))
    w = dev(rng.normal(size=grid.N))
    pts = dev(rng.uniform(-0.5, nx * res + 0.5, size=(LIMIT + 1, 2))).to(dtype)
    full = ctx.eval(p, grid, w, pts)
    bits = torch.int32 if dtype == torch.float32 else torch.int64
    last = min(lim // grid.max_candidates - 2000, LIMIT)
    assert 1000 < last
    for Q in (last, last + 1):
        part = ctx.eval(p, grid, w, pts[:Q])
        for key in ("f", "grad"):
            assert torch.equal(part[key].view(bits), full[key][:Q].view(bits)), (Q, key)
