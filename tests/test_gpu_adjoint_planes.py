"""Adjoint with the weights' gradient summed in LDS planes, on both sides of
its rules (centers that fit, points per plane), against the sum of calls too
small for it, which add with device atomics.

Tolerance: both add the same terms a_i phi_ij (a term is formed by the same
operations) in another order, so an entry differs by at most 2 Q eps times the
sum of its terms' absolute values, which a call with |a_i| gives."""
import numpy as np
import pytest
import torch

from helpers import dev, host
from paper_2509_26222_amd import api, synth

pytestmark = pytest.mark.gpu
EPS = np.finfo(np.float64).eps
SMALL = 4095  # largest call that adds with device atomics


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("n,extra,Q", [(20, 0, 4095), (20, 0, 4096), (20, 0, 4353),
                                       (134, 0, 70001), (192, 0, 36863), (192, 0, 36864),
                                       (192, 1, 36866)])
def test_planes_match_atomics(ctx, dtype, dim, n, extra, Q):
    p = api.Params()
    rng = np.random.default_rng(n + Q)
    ny = 96 if n == 192 else n
    c = synth.grid_centers(rng, n, ny, 0.5, jitter=0.1)
    c = np.concatenate([c, c[:extra] + 0.2])
    grid = ctx.grid(p, dev(c))
    w = dev(rng.normal(size=c.shape[0]))
    xyz = np.concatenate([rng.uniform(-1.0, [0.5 * n + 1.0, 0.5 * ny + 1.0], size=(Q, 2)),
                          rng.normal(size=(Q, 1))], 1)
    xyz[: Q // 4, :2] = [3.1, 3.2] + 0.01 * xyz[: Q // 4, :2]  # many on few centers
    pts = dev(xyz[:, :dim]).to(dtype).contiguous()
    gf = dev(rng.normal(size=Q)).to(dtype)
    gf[5:9] = 0
    pose = (synth.rot_zyx(0.3, 0.02, -0.01), np.array([0.1, -0.2, 0.3])) if dim == 3 else None
    gr = dev(rng.normal(size=Q)).to(dtype) if dim == 3 else None

    def call(sl, g, r, d_w):
        d_pose = torch.zeros(6, dtype=torch.float64, device="cuda") if dim == 3 else None
        dp, _, _ = ctx.eval_adjoint(p, grid, w, pts[sl], pose=pose, gbar_f=g[sl],
                                    gbar_r=None if r is None else r[sl], d_w=d_w, d_pose=d_pose)
        return dp, d_pose

    start = dev(rng.normal(size=c.shape[0]))
    got = start.clone()
    dp, dpose = call(slice(0, Q), gf, gr, got)
    ref, parts, poses = start.clone(), [], []
    for s in range(0, Q, SMALL):
        a, b = call(slice(s, min(s + SMALL, Q)), gf, gr, ref)
        parts.append(a)
        poses.append(b)
    assert torch.equal(dp, torch.cat(parts))
    a = gf if gr is None else gf - gr
    mag = torch.zeros_like(start)
    for s in range(0, Q, SMALL):
        call(slice(s, min(s + SMALL, Q)), a.abs(), None, mag)
    tol = host(mag + start.abs()) * 2 * (Q + 1) * EPS
    assert np.all(np.abs(host(got) - host(ref)) <= tol)
    if dim == 3:
        size = torch.cat([q.abs().to(torch.float64) for q in parts]).sum()
        lim = 4 * Q * EPS * float(size) * (1.0 + float(pts.abs().max()))
        assert np.all(np.abs(host(dpose) - host(sum(poses))) <= lim)


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("res,nx,ny,Q", [(0.5, 20, 17, 4096), (0.5, 100, 60, 20_011),
                                         (1.0, 30, 30, 5000), (0.3, 25, 25, 5000),
                                         (0.5, 128, 120, 31_000), (0.5, 128, 121, 31_000)])
def test_mesh_planes(ctx, dim, res, nx, ny, Q):
    """FP64 on a mesh: windows of 8, 4 and 12 nodes (the last by the binned
    form), node arrays that fit (144 x 128 = 18,432 nodes and margins) and not.
    Against the atomics of small calls: the terms agree to rounding, a value's
    exponent (at most cutoff^2 / 2 <= 5) to 8 eps on either side, so a term to
    100 eps, a sum of at most Q terms to (2 Q + 100) eps of its absolute sum."""
    p = api.Params()
    rng = np.random.default_rng(nx + Q)
    c = synth.grid_centers(rng, nx, ny, res, jitter=0.0)
    keep = rng.random(c.shape[0]) < 0.9
    keep[[0, -1]] = True
    c = np.ascontiguousarray(c[keep])
    grid = ctx.grid(p, dev(c)).set_mesh_roi((0.0, 0.0), res)
    w = dev(rng.normal(size=c.shape[0]))
    xyz = np.concatenate([rng.uniform(-2.0, [nx * res + 2.0, ny * res + 2.0], size=(Q, 2)),
                          rng.normal(size=(Q, 1))], 1)
    xyz[3, 0], xyz[4, 1] = 1e30, -1e9
    pts = dev(xyz[:, :dim]).contiguous()
    pose = (synth.rot_zyx(0.3, 0.02, -0.01), np.array([0.1, -0.2, 0.3])) if dim == 3 else None
    gf = dev(rng.normal(size=Q))
    gf[5:9] = 0
    gr = dev(rng.normal(size=Q)) if dim == 3 else None

    def call(sl, wt, g, r, d_w):
        d_pose = torch.zeros(6, dtype=torch.float64, device="cuda") if dim == 3 else None
        dp, _, _ = ctx.eval_adjoint(p, grid, wt, pts[sl], pose=pose, gbar_f=g[sl],
                                    gbar_r=None if r is None else r[sl], d_w=d_w, d_pose=d_pose)
        return dp, d_pose

    def small(wt, g, r):
        d_w, parts, poses = torch.zeros_like(w), [], 0
        for s in range(0, Q, SMALL):
            a, b = call(slice(s, min(s + SMALL, Q)), wt, g, r, d_w)
            parts.append(a)
            poses = poses + b if dim == 3 else None
        return d_w, torch.cat(parts), poses

    got = torch.zeros_like(w)
    dp, dpose = call(slice(0, Q), w, gf, gr, got)
    ref, rp, rpose = small(w, gf, gr)
    a = gf if gr is None else gf - gr
    mag, _, _ = small(w, a.abs(), None)
    tol = (2 * Q + 100) * EPS
    assert np.all(np.abs(host(got) - host(ref)) <= tol * host(mag) + 1e-300)
    # a point's gradient: at most 144 nodes of |w| phi |dx| / sigma^2
    size = float(a.abs().max()) * 144 * float(w.abs().max()) * p.cutoff / p.sigma
    assert float((dp - rp).abs().max()) <= 4 * 300 * EPS * (size + 1.0)
    if dim == 3:
        reach = 1.0 + float(pts[5:].abs().max())
        far = pts[3:5].abs().sum() * (float(gr[3:5].abs().max()) + 1.0)
        lim = Q * 4 * 300 * EPS * (size + 4.0) * reach + 16 * EPS * float(far)
        assert np.all(np.abs(host(dpose) - host(rpose)) <= lim)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("n,Q", [(30, 4200), (30, 4400), (70, 12_500), (70, 14_000)])
def test_both_sides_of_the_additions_rule(ctx, dtype, n, Q):
    test_planes_match_atomics(ctx, dtype, 3, n, 0, Q)


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("Q", [15_000, 16_500])
def test_mesh_planes_of_sparse_centers(ctx, dim, Q):
    """Windows of 4 nodes, seven centers in a support: on both sides of the rule."""
    test_mesh_planes(ctx, dim, 1.0, 30, 30, Q)
