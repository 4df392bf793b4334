"""The work that a user of the terrain library has it do, as timed cases.

A case is one call, or the few calls of one step of a mapping program, on
synthetic terrain: smooth bumps with 2 cm height noise, centers 0.5 m apart
(sigma 0.5 m, cutoff 3, lambda 1e-3), points in a disc around the sensor as
a scan gives them. `kind` says which step:

  eval     height, gradient (and, at body-frame points, residual and pose
           Jacobian) at scan points
  gn       the fused Gauss-Newton sums of one pose iteration
  adjoint  the backward pass: gradients for points, weights and pose
  update   one scan absorbed by the recursive update (sort, then update)
  mixed    the same with low-precision covariance products, the information
           form accumulated beside it and the weights refined against it
  solve    the whole map from its information form: assembly, sparse solve
  patches  many uneven patches, updated and evaluated by one plan
  build    a new map: center selection, binning, the first scan sorted
"""
import math

import numpy as np
import torch

from paper_2509_26222_amd import api

RES = 0.5     # center spacing, metres
SIGMA = 0.5
CUTOFF = 3.0
LAM = 1e-3
R_VAR = 0.02 ** 2
NOISE = 0.02  # std of the ground heights
DEV = "cuda:0"
F64 = torch.float64
DT = {"f32": torch.float32, "f64": torch.float64}
PARAMS = api.Params(sigma=SIGMA, cutoff=CUTOFF, sigma_eps=0.0, lam=LAM, R=R_VAR)

_ctx = []


def ctx():
    """The program's one context."""
    if not _ctx:
        _ctx.append(api.Context(0))
    return _ctx[0]


# ------------------------------------------------------------------- cases

def listed():
    return [
        # a few foothold queries against a small jittered map: latency only
        dict(name="eval_xy_small", kind="eval", nx=20, ny=20, mesh=False, Q=1000, dim=2,
             dtype="f64"),
        # one scan on the odometry map (10,000 mesh centers), the form that
        # runs at every frame
        dict(name="eval_scan_f32", kind="eval", nx=100, ny=100, mesh=True, Q=200_000, dim=3,
             dtype="f32"),
        # half a scan in double precision on centers that lie on no mesh
        dict(name="eval_binned_f64", kind="eval", nx=99, ny=101, mesh=False, Q=100_003, dim=3,
             dtype="f64"),
        # a whole session's points at once (map quality check, re-projection)
        dict(name="eval_map_f32", kind="eval", nx=100, ny=100, mesh=True, Q=5_000_000, dim=3,
             dtype="f32"),
        # one Gauss-Newton iteration of the pose against one scan
        dict(name="gn_scan_f32", kind="gn", nx=100, ny=100, mesh=True, Q=200_000, dtype="f32"),
        # backward of one scan's heights and residuals (learning, smoothing)
        dict(name="adjoint_scan_f64", kind="adjoint", nx=100, ny=100, mesh=True, Q=200_000,
             dtype="f64"),
        # one recursive update of a 10 x 10 m patch, default batch
        dict(name="update_small", kind="update", nx=20, ny=20, M=2000, batch=0),
        # one odometry frame: 20,000 ground points into 10,000 centers
        dict(name="update_frame", kind="update", nx=100, ny=100, M=20_000, batch=1024),
        # a frame of a middle-sized map with BF16x3 products and refinement
        dict(name="mixed_bf16", kind="mixed", nx=71, ny=71, M=10_007, batch=1024,
             prec="bf16"),
        # a 100 x 100 m map solved from 800,000 points (plan kept)
        dict(name="solve_map_40k", kind="solve", nx=200, ny=200, M=800_000),
        # 24 uneven patches in one graph launch
        dict(name="patches_24", kind="patches", count=24, n_lo=200, n_hi=2000, m_lo=1000,
             m_hi=6000),
        # a new 50 x 50 m map from the points of a whole session
        dict(name="build_map", kind="build", nx=100, ny=100, M=2_000_000, mode="radius"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["eval", "eval", "eval", "gn", "adjoint", "update", "update", "mixed",
                       "solve", "patches", "build"])
    if kind in ("eval", "gn", "adjoint"):
        c = dict(kind=kind, nx=rng.randint(15, 110), ny=rng.randint(15, 110),
                 mesh=rng.random() < 0.6,
                 Q=_log(rng, 200, 5_000_000 if kind == "eval" else 400_000),
                 dtype=rng.choice(["f32", "f64"]))
        if kind == "eval":
            c["dim"] = rng.choice([2, 3, 3])
            if c["dtype"] == "f64":
                c["Q"] = min(c["Q"], 2_000_000 + rng.randint(0, 99))
        return c
    if kind == "update":
        return dict(kind=kind, nx=rng.randint(14, 99), ny=rng.randint(14, 99),
                    M=_log(rng, 300, 18_000), batch=rng.choice([0, 512, 1024, 2048]))
    if kind == "mixed":
        return dict(kind=kind, nx=rng.randint(25, 75), ny=rng.randint(25, 75),
                    M=_log(rng, 1000, 12_000), batch=1024, prec=rng.choice(["f32", "bf16"]))
    if kind == "solve":
        return dict(kind=kind, nx=rng.randint(30, 200), ny=rng.randint(30, 200),
                    M=_log(rng, 20_000, 800_000))
    if kind == "patches":
        return dict(kind=kind, count=rng.randint(4, 24), n_lo=200, n_hi=rng.randint(600, 2000),
                    m_lo=1000, m_hi=rng.randint(1500, 6000))
    return dict(kind=kind, nx=rng.randint(20, 110), ny=rng.randint(20, 110),
                M=_log(rng, 20_000, 2_000_000), mode=rng.choice(["radius", "voxel"]))


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, dtype=F64, device=DEV)


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, dtype=F64, device=DEV)


def _lattice(nx, ny):
    """Cell centers of the candidate mesh, row-major (y outer)."""
    i = (torch.arange(nx, dtype=F64, device=DEV) + 0.5) * RES
    j = (torch.arange(ny, dtype=F64, device=DEV) + 0.5) * RES
    return torch.stack([i.repeat(ny), j.repeat_interleave(nx)], 1).contiguous()


def _centers(g, nx, ny, mesh):
    c = _lattice(nx, ny)
    return c if mesh else c + (_rand(g, nx * ny, 2) - 0.5) * 0.2


def _bumps(g, w, h):
    k = 40
    lo = torch.tensor([w, h], dtype=F64, device=DEV)
    return _rand(g, k, 2) * lo, (_rand(g, k) - 0.5) * 0.4, 0.3 + 1.2 * _rand(g, k)


def _height(t, xy):
    mu, a, s = t
    z = torch.zeros(xy.shape[0], dtype=F64, device=DEV)
    for k in range(mu.shape[0]):
        z += a[k] * torch.exp(-((xy - mu[k]) ** 2).sum(1) / (2 * s[k] ** 2))
    return z


def _disc(g, n, w, h):
    """n points uniform in a 20 m disc around the sensor, clipped to the map."""
    at = [float(v) for v in (0.3 + 0.4 * _rand(g, 2)).cpu()]
    cx, cy = at[0] * w, at[1] * h
    rad = min(20.0, 0.6 * max(w, h))
    got, have = [], 0
    while have < n:
        k = int((n - have) * 2.2) + 256
        r, th = rad * torch.sqrt(_rand(g, k)), 2 * math.pi * _rand(g, k)
        p = torch.stack([cx + r * torch.cos(th), cy + r * torch.sin(th)], 1)
        p = p[(p[:, 0] >= 0) & (p[:, 0] < w) & (p[:, 1] >= 0) & (p[:, 1] < h)]
        got.append(p)
        have += p.shape[0]
    return torch.cat(got)[:n].contiguous(), (cx, cy)


def _rot(yaw, pitch, roll):
    cy, sy, cp, sp = math.cos(yaw), math.sin(yaw), math.cos(pitch), math.sin(pitch)
    cr, sr = math.cos(roll), math.sin(roll)
    rz = np.array([[cy, -sy, 0], [sy, cy, 0], [0, 0, 1.0]])
    ry = np.array([[cp, 0, sp], [0, 1.0, 0], [-sp, 0, cp]])
    rx = np.array([[1.0, 0, 0], [0, cr, -sr], [0, sr, cr]])
    return rz @ ry @ rx


def _scan(case, seed):
    """Centers, fitted-looking weights, scan points and pose."""
    g = _gen(seed)
    nx, ny = case["nx"], case["ny"]
    w_, h_ = nx * RES, ny * RES
    c = _centers(g, nx, ny, case["mesh"])
    t = _bumps(g, w_, h_)
    # heights divided by the kernel's sum over the mesh, and the scatter of
    # a fit to noisy points
    w = _height(t, c) * (RES * RES / (2 * math.pi * SIGMA ** 2)) + 0.02 * _randn(g, nx * ny)
    xy, (sx, sy) = _disc(g, case["Q"], w_, h_)
    if case.get("dim", 3) == 2:
        return c, w, xy.to(DT[case["dtype"]]).contiguous(), None
    z = _height(t, xy) + NOISE * _randn(g, case["Q"])
    a = [float(v) for v in _rand(g, 3).cpu()]
    R = _rot(2 * math.pi * a[0], math.radians(10 * a[1] - 5), math.radians(10 * a[2] - 5))
    tr = np.array([sx, sy, 0.6])
    world = torch.cat([xy, z[:, None]], 1)
    body = (world - torch.tensor(tr, device=DEV)) @ torch.tensor(R, device=DEV)
    return c, w, body.to(DT[case["dtype"]]).contiguous(), (R, tr)


def _ground(case, seed, whole=False):
    """Centers (mesh), ground points and noisy heights: a disc around the
    sensor, or the whole map."""
    g = _gen(seed)
    w_, h_ = case["nx"] * RES, case["ny"] * RES
    c = _lattice(case["nx"], case["ny"])
    t = _bumps(g, w_, h_)
    if whole:
        xy = _rand(g, case["M"], 2) * torch.tensor([w_, h_], dtype=F64, device=DEV)
    else:
        xy, _ = _disc(g, case["M"], w_, h_)
    return c, xy, _height(t, xy) + NOISE * _randn(g, case["M"])


def _patch_inputs(case, seed):
    """Per patch: its mesh, jittered centers, points, heights. The sizes are
    the case's, the terrain and the points the seed's."""
    rs = np.random.default_rng([case["count"], case["n_hi"], case["m_hi"]])
    g = _gen(seed)
    out = []
    for _ in range(case["count"]):
        n = int(rs.integers(case["n_lo"], case["n_hi"] + 1))
        m = int(rs.integers(case["m_lo"], case["m_hi"] + 1))
        nx = int(round(math.sqrt(n)))
        ny = n // nx
        w_, h_ = nx * RES, ny * RES
        c = _centers(g, nx, ny, False)
        t = _bumps(g, w_, h_)
        xy = _rand(g, m, 2) * torch.tensor([w_, h_], dtype=F64, device=DEV)
        out.append((nx, ny, c, xy, _height(t, xy) + NOISE * _randn(g, m)))
    return out


def _prior(n):
    P = torch.zeros((n, n), dtype=F64, device=DEV)
    P.diagonal().fill_(R_VAR / LAM)
    return torch.zeros(n, dtype=F64, device=DEV), P


# ------------------------------------------------------------ prepare, run

def prepare(case, seed):
    k = case["kind"]
    cx = ctx()
    s = {"case": case, "ctx": cx}
    if k in ("eval", "gn", "adjoint"):
        c, s["w"], s["pts"], s["pose"] = _scan(case, seed)
        s["grid"] = cx.grid(PARAMS, c)
        if case["mesh"]:
            s["grid"].set_mesh_roi((0.0, 0.0), RES)
        if k == "adjoint":
            g = _gen(seed + 1)
            s["gf"] = _randn(g, case["Q"]).to(s["pts"].dtype)
            s["gr"] = _randn(g, case["Q"]).to(s["pts"].dtype)
    elif k in ("update", "mixed"):
        c, s["xy"], s["z"] = _ground(case, seed)
        s["grid"] = cx.grid(PARAMS, c)
        s["w"], s["P"] = _prior(c.shape[0])
        if k == "mixed":
            s["rowptr"], s["colidx"] = cx.gram_pattern(PARAMS, s["grid"])
            s["vals"] = torch.zeros(s["colidx"].shape[0], dtype=F64, device=DEV)
            s["b"] = torch.zeros(c.shape[0], dtype=F64, device=DEV)
            s["first"] = True
    elif k == "solve":
        c, s["xy"], s["z"] = _ground(case, seed, whole=True)
        s["grid"] = cx.grid(PARAMS, c)
        s["rowptr"], s["colidx"] = cx.gram_pattern(PARAMS, s["grid"])
        s["plan"] = cx.solve_plan(s["rowptr"], s["colidx"])
    elif k == "patches":
        raw = _patch_inputs(case, seed)
        ns, ms = [p[2].shape[0] for p in raw], [p[3].shape[0] for p in raw]
        q = sum(ms)
        f32 = dict(dtype=torch.float32, device=DEV)
        out = {"w": torch.zeros(sum(ns), dtype=F64, device=DEV),
               "P": torch.zeros(sum(n * n for n in ns), dtype=F64, device=DEV),
               "f": torch.empty(q, **f32), "grad": torch.empty((q, 2), **f32),
               "resid": torch.empty(q, **f32), "jac": torch.empty((q, 6), **f32)}
        patches, a, b, e = [], 0, 0, 0
        for (nx, ny, c, xy, z), n, m in zip(raw, ns, ms):
            grid = cx.grid(PARAMS, c)
            xs, zs, _ = cx.sort_points(grid, xy, z)
            P = out["P"][b:b + n * n].view(n, n)
            P.diagonal().fill_(R_VAR / LAM)
            patches.append(dict(grid=grid, w=out["w"][a:a + n], P=P, xy=xs, z=zs,
                                pts=torch.cat([xs, zs[:, None]], 1).float().contiguous(),
                                pose=(np.eye(3), np.zeros(3)), f=out["f"][e:e + m],
                                grad=out["grad"][e:e + m], resid=out["resid"][e:e + m],
                                jac=out["jac"][e:e + m]))
            a, b, e = a + n, b + n * n, e + m
        s["out"] = out
        s["plan"] = api.Batched(cx, PARAMS, patches, dim=3, eval_prec="f32", gemm_prec="f64")
    else:
        _, s["xy"], _ = _ground(case, seed, whole=True)
        m = min(20_000, case["M"])
        s["scan_xy"] = s["xy"][:m].contiguous()
        s["scan_z"] = _randn(_gen(seed + 2), m)
    return s


def run(s):
    case, cx = s["case"], s["ctx"]
    k = case["kind"]
    if k == "eval":
        return cx.eval(PARAMS, s["grid"], s["w"], s["pts"], pose=s["pose"])
    if k == "gn":
        return cx.eval_gn(PARAMS, s["grid"], s["w"], s["pts"], s["pose"])
    if k == "adjoint":
        d_w = torch.zeros_like(s["w"])
        d_pose = torch.zeros(6, dtype=F64, device=DEV)
        return cx.eval_adjoint(PARAMS, s["grid"], s["w"], s["pts"], pose=s["pose"],
                               gbar_f=s["gf"], gbar_r=s["gr"], d_w=d_w, d_pose=d_pose)
    if k == "update":
        xs, zs, _ = cx.sort_points(s["grid"], s["xy"], s["z"])
        cx.update(PARAMS, s["grid"], s["w"], s["P"], xs, zs, batch=case["batch"])
        return {"w": s["w"], "P": s["P"]}
    if k == "mixed":
        xs, zs, _ = cx.sort_points(s["grid"], s["xy"], s["z"])
        cx.update(PARAMS, s["grid"], s["w"], s["P"], xs, zs, batch=case["batch"],
                  gemm_prec=case["prec"])
        cx.assemble_gram(PARAMS, s["grid"], xs, zs, s["rowptr"], s["colidx"], s["vals"],
                         s["b"], add_lambda=s["first"])
        s["first"] = False  # lambda is added once
        cx.refine(PARAMS, s["rowptr"], s["colidx"], s["vals"], s["b"], s["P"], s["w"],
                  rtol=1e-10, max_iter=30)
        return {"w": s["w"], "P": s["P"], "vals": s["vals"], "b": s["b"]}
    if k == "solve":
        vals, b = cx.assemble_gram(PARAMS, s["grid"], s["xy"], s["z"], s["rowptr"], s["colidx"])
        x, _, _, _ = s["plan"].run(vals, b, rtol=1e-10)
        return {"vals": vals, "b": b, "x": x}
    if k == "patches":
        s["plan"].run()
        s["plan"].sync()
        return s["out"]
    roi = (0.0, 0.0, case["nx"] * RES, case["ny"] * RES)
    mode = api.L.SELECT_RADIUS if case["mode"] == "radius" else api.L.SELECT_VOXEL
    centers = cx.select_centers(s["xy"], roi, RES, 0.5, 4, mode)
    grid = cx.grid(PARAMS, centers).set_mesh_roi(roi, RES)
    xs, zs, perm = cx.sort_points(grid, s["scan_xy"], s["scan_z"])
    grid.close()
    return {"centers": centers, "xy": xs, "z": zs, "perm": perm}


# -------------------------------------------------------------------- work

def work(case):
    """Inputs read once, outputs written once; the operations of the step
    itself (28 centers in a point's support)."""
    k = case["kind"]
    if k in ("eval", "gn", "adjoint"):
        q, n, e = case["Q"], case["nx"] * case["ny"], 8 if case["dtype"] == "f64" else 4
        dim = case.get("dim", 3)
        if k == "eval":
            per = (2 + 3) * e if dim == 2 else (3 + 10) * e
        else:
            per = 3 * e if k == "gn" else (3 + 2 + 3) * e
        return {"bytes": q * per + 8 * n * (2 if k == "adjoint" else 1), "flops": q * 28 * 10}
    if k in ("update", "mixed"):
        n, m = case["nx"] * case["ny"], case["M"]
        # the part of P - V V^T that symmetry leaves, of rank min(M, N)
        nnz = 113 * n if k == "mixed" else 0
        return {"bytes": 16 * n * n + 24 * m + 16 * n + 16 * nnz,
                "flops": n * (n + 1) * min(m, n)}
    if k == "solve":
        n, m = case["nx"] * case["ny"], case["M"]
        return {"bytes": 16 * 113 * n + 24 * m + 16 * n,
                "flops": m * 28 * 28 * 2 + 3.6e10 * (n / 4e4) ** 1.5}
    if k == "patches":
        n, m = (case["n_lo"] + case["n_hi"]) / 2, (case["m_lo"] + case["m_hi"]) / 2
        return {"bytes": case["count"] * (16 * n * n + m * (24 + 52)),
                "flops": case["count"] * (n * n * min(m, n) + m * 280)}
    m = min(20_000, case["M"])
    return {"bytes": 16 * case["M"] + 52 * m + 16 * case["nx"] * case["ny"],
            "flops": case["M"] * 30}


# ------------------------------------------------------------------- exact

def _window(xy, c, nx, ny):
    """Around each point the 8 x 8 centers that can lie in its support: their
    indices, kernel values and offsets x - c (zero where out of the support)."""
    k = torch.arange(-4, 4, device=DEV)
    i = torch.floor(xy[:, 0] / RES).long()[:, None] + k
    j = torch.floor(xy[:, 1] / RES).long()[:, None] + k
    ok = (((j >= 0) & (j < ny))[:, :, None] & ((i >= 0) & (i < nx))[:, None, :]).flatten(1)
    idx = (j.clamp(0, ny - 1)[:, :, None] * nx + i.clamp(0, nx - 1)[:, None, :]).flatten(1)
    d = xy[:, None, :] - c[idx]
    d2 = (d * d).sum(2)
    phi = torch.exp(-d2 / (2 * SIGMA ** 2)) * (ok & (d2 <= (CUTOFF * SIGMA) ** 2))
    return idx, phi, d


def _model(xy, c, w, nx, ny):
    idx, phi, d = _window(xy, c, nx, ny)
    pw = phi * w[idx]
    return idx, phi, pw.sum(1), -(pw[:, :, None] * d).sum(1) / SIGMA ** 2


def _terms(pts, pose, c, w, nx, ny):
    """Per point: window, kernel values, f, grad f, residual, Jacobian."""
    R, t = (torch.tensor(np.asarray(v), dtype=F64, device=DEV) for v in pose)
    xi = pts @ R.T + t
    idx, phi, f, grad = _model(xi[:, :2], c, w, nx, ny)
    g = torch.cat([-grad, torch.ones_like(f)[:, None]], 1)
    J = torch.cat([torch.linalg.cross(pts, g @ R), g], 1)
    return R, idx, phi, f, grad, xi[:, 2] - f, J


def _chunks(n, size=100_000):
    return [(a, min(a + size, n)) for a in range(0, n, size)]


def _rows(xy, c, nx, ny):
    """The regressor rows of the points, dense (M x N)."""
    H = torch.zeros((xy.shape[0], c.shape[0]), dtype=F64, device=DEV)
    idx, phi, _ = _window(xy, c, nx, ny)
    # an index of a clamped place comes with phi = 0 and may repeat: add
    return H.scatter_add_(1, idx, phi)


def _ridge(c, xy, z, nx, ny):
    H = _rows(xy, c, nx, ny)
    A = H.T.contiguous() @ H
    b = H.T @ z
    A.diagonal().add_(LAM)
    L = torch.linalg.cholesky(A)
    inv = torch.cholesky_inverse(L)
    w = torch.cholesky_solve(b[:, None], L)[:, 0]
    return A, b, w, R_VAR * inv


def _pattern(nx, ny):
    """Rows and columns of the mesh's Gram pattern (centers closer than two
    support radii), columns ascending within a row."""
    r = int(2 * CUTOFF * SIGMA / RES)
    off = [(dj, di) for dj in range(-r, r + 1) for di in range(-r, r + 1)
           if dj * dj + di * di <= r * r]
    i = torch.arange(nx, device=DEV).repeat(ny)[:, None]
    j = torch.arange(ny, device=DEV).repeat_interleave(nx)[:, None]
    dj = torch.tensor([o[0] for o in off], device=DEV)
    di = torch.tensor([o[1] for o in off], device=DEV)
    ok = (i + di >= 0) & (i + di < nx) & (j + dj >= 0) & (j + dj < ny)
    col = (j + dj) * nx + i + di
    row = torch.arange(nx * ny, device=DEV)[:, None].expand_as(col)
    return row[ok], col[ok]


def exact(case, seed):
    k = case["kind"]
    if k == "patches":
        got = {n: [] for n in ("w", "P", "f", "grad", "resid", "jac")}
        for nx, ny, c, xy, z in _patch_inputs(case, seed):
            _, _, w, P = _ridge(c, xy, z, nx, ny)
            got["w"].append(w)
            got["P"].append(P.reshape(-1))
            # the plan's points are in the order of its bins: not known here
        return {n: torch.cat(v) if v else None for n, v in got.items()}
    nx, ny = case["nx"], case["ny"]
    if k in ("eval", "gn", "adjoint"):
        c, w, pts, pose = _scan(case, seed)
        pts = pts.double()
        if k == "eval":
            parts = []
            for a, b in _chunks(case["Q"]):
                if pose is None:
                    _, _, f, grad = _model(pts[a:b], c, w, nx, ny)
                    parts.append((f, grad))
                else:
                    _, _, _, f, grad, r, J = _terms(pts[a:b], pose, c, w, nx, ny)
                    parts.append((f, grad, r, J))
            parts = [torch.cat(p) for p in zip(*parts)] + [None, None]
            return dict(zip(("f", "grad", "resid", "jac"), parts))
        if k == "gn":
            JJ, Jr, rr = 0, 0, 0
            for a, b in _chunks(case["Q"]):
                _, _, _, _, _, r, J = _terms(pts[a:b], pose, c, w, nx, ny)
                Jt = J.T.contiguous()
                JJ, Jr, rr = JJ + Jt @ J, Jr + Jt @ r, rr + (r * r).sum()
            return JJ, Jr, rr
        g = _gen(seed + 1)
        dt = DT[case["dtype"]]
        gf, gr = _randn(g, case["Q"]).to(dt).double(), _randn(g, case["Q"]).to(dt).double()
        d_pts, d_w, d_pose = [], torch.zeros_like(w), torch.zeros(6, dtype=F64, device=DEV)
        for a, b in _chunks(case["Q"]):
            R, idx, phi, _, grad, _, _ = _terms(pts[a:b], pose, c, w, nx, ny)
            al = gf[a:b] - gr[a:b]
            d_xi = torch.cat([al[:, None] * grad, gr[a:b, None]], 1)
            d_p = d_xi @ R
            d_pts.append(d_p)
            d_w.index_add_(0, idx.reshape(-1), (phi * al[:, None]).reshape(-1))
            d_pose += torch.cat([torch.linalg.cross(pts[a:b], d_p), d_xi], 1).sum(0)
        return torch.cat(d_pts), d_w, d_pose
    if k in ("update", "mixed"):
        c, xy, z = _ground(case, seed)
        A, b, w, P = _ridge(c, xy, z, nx, ny)
        if k == "update":
            return {"w": w, "P": P}
        row, col = _pattern(nx, ny)
        return {"w": w, "P": P, "vals": A[row, col], "b": b}
    if k == "solve":
        c, xy, z = _ground(case, seed, whole=True)
        n = nx * ny
        A = torch.zeros(n * n, dtype=F64, device=DEV)
        b = torch.zeros(n, dtype=F64, device=DEV)
        for a, e in _chunks(case["M"], 20_000):
            idx, phi, _ = _window(xy[a:e], c, nx, ny)
            A.index_add_(0, (idx[:, :, None] * n + idx[:, None, :]).reshape(-1),
                         (phi[:, :, None] * phi[:, None, :]).reshape(-1))
            b.index_add_(0, idx.reshape(-1), (phi * z[a:e, None]).reshape(-1))
        A = A.view(n, n)
        row, col = _pattern(nx, ny)
        vals = A[row, col]
        A.diagonal().add_(LAM)
        vals = vals + LAM * (row == col)
        L = torch.linalg.cholesky(A)
        return {"vals": vals, "b": b, "x": torch.cholesky_solve(b[:, None], L)[:, 0]}
    # selection: exact counts; the order of sorted points is the grid's own
    _, xy, _ = _ground(case, seed, whole=True)
    G = _lattice(nx, ny)
    cnt = torch.zeros(nx * ny, dtype=torch.int64, device=DEV)
    ij = torch.floor(xy / RES).long()
    for dj in (-1, 0, 1):
        for di in (-1, 0, 1):
            i, j = ij[:, 0] + di, ij[:, 1] + dj
            ok = (i >= 0) & (i < nx) & (j >= 0) & (j < ny)
            node = j.clamp(0, ny - 1) * nx + i.clamp(0, nx - 1)
            if case["mode"] == "radius":
                ok &= ((xy - G[node]) ** 2).sum(1) <= 0.25
            else:
                ok &= (di == 0) & (dj == 0)
            cnt.index_add_(0, node, ok.long())
    return {"centers": G[cnt > 4], "xy": None, "z": None, "perm": None}
