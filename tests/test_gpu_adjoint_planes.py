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
