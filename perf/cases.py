"""Performance cases of the bundle-adjustment library.

Each case is one call, or one short sequence of calls, that a program built on
`paper_2307_08383_amd.ba` makes over and over: an LM step, the four calls of a
caller's own LM loop, a solve with a formed reduced camera system (RCS),
re-triangulation, and the cost of a set of parameters.  The scenes are the
ones of the repository's tests and benchmark (nadir blocks of 16 to 60,000
cameras, mean track length 4, a few tens of co-visible cameras each), made on
the GPU from the case's seed.

`op` of a case:
  step         ba_lm_step on a context of 9-parameter cameras
  shared_step  ba_lm_step on a shared-intrinsics context
  solve        ba_linearize, ba_form_rcs, ba_pcg_solve, ba_back_substitute
  retry        ba_form_rcs with another damping, ba_pcg_solve and
               ba_back_substitute on a linearization that stays (what follows
               a rejected step)
  pcg          ba_pcg_solve on a formed RCS
  triangulate  ba_triangulate, linear start and Gauss-Newton steps
  cost         ba_cost_noalloc

Solves on large scenes stop at an iteration cap (an inexact step, as the
benchmark's capped solves); on smaller ones and with the factorised
preconditioners they run to a tolerance.
"""
import math

import numpy as np
import torch

from paper_2307_08383_amd import ba

DEV = "cuda"
F64 = torch.float64

# Mean track length: truncated geometric on [2, 12] (P(t) ~ Q ** (t - 2)).
Q_TRACK = 0.71
LONG_FROM = 65        # distant points are seen by at least this many cameras


def listed():
    base = dict(nx=4, ny=4, ring=0, step_x=1.0, nearest=True, n_pts=500, n_long=0, n_phys=0, precision="fp64",
                precond="block_jacobi", deflate=False, solver_fp32=False, lam=1e-4, tol=1e-6, max_iter=1000)

    def case(name, op, **kw):
        c = dict(base, name=name, op=op)
        c.update(kw)
        return c

    return [
        # The smallest problem (16 cameras, 500 points): an LM step, where launches and latency count; small local
        # adjustments run many of these.
        case("step_tiny", "step", nx=4, ny=4, n_pts=500, tol=1e-10),
        # An 80-image block flown with 4 physical cameras that share their interior unknowns.
        case("shared_step_block", "shared_step", nx=10, ny=8, n_pts=20_000, n_phys=4, lam=1e-2, tol=1e-10),
        # 300 cameras with a few landmarks that a large part of the block sees (tracks longer than 64),
        # factorised preconditioner.
        case("step_block_fsai_long", "step", nx=20, ny=15, n_pts=60_011, n_long=4, precond="fsai", lam=1e-3,
             tol=1e-10),
        # The 2,000-camera aerial block of the tests and the benchmark, an LM step to the default tolerance.
        case("step_aerial", "step", nx=50, ny=40, n_pts=400_000, lam=1e-3),
        # The same block after a rejected step, FP32 records: formation with a heavier damping and the solve.
        case("retry_aerial_mixed", "retry", nx=45, ny=37, n_pts=333_333, precision="mixed", lam=1e-3, max_iter=50),
        # Solve of the aerial block's RCS with the exact factorised preconditioner and the gauge deflated.
        case("pcg_aerial_fsai", "pcg", nx=50, ny=40, n_pts=400_000, precond="fsai", deflate=True, lam=1e-3,
             tol=1e-12),
        # A caller's own LM loop on a quarter of the benchmark's partition, FP64: formation carries it.
        case("solve_partition", "solve", nx=125, ny=120, ring=2, nearest=False, n_pts=6_250_000, max_iter=8),
        # Flight strips (80% forward overlap), FP32 records and solver matrix: an inexact LM step.
        case("step_strips_mixed", "step", nx=3600, ny=5, step_x=0.5, n_pts=4_500_000, precision="mixed",
             solver_fp32=True, max_iter=30),
        # The benchmark's 60,000-camera partition (its RCS; fewer points a camera): the solve that an LM step
        # spends most of its time in, the paper's preconditioner.
        case("pcg_partition", "pcg", nx=250, ny=240, ring=2, nearest=False, n_pts=3_000_000, max_iter=64),
        # The learned factorised preconditioner on half of that partition, mixed precision, gauge deflated: the
        # network runs on the new RCS, then the solve.
        case("retry_partition_learned", "retry", nx=175, ny=170, ring=2, nearest=False, n_pts=2_000_000,
             precision="mixed", precond="learned_fsai", deflate=True, lam=1e-2, tol=1e-12),
        # All points of a strip block re-triangulated with the cameras fixed.
        case("triangulate_strips", "triangulate", nx=1800, ny=5, step_x=0.5, n_pts=2_250_000, max_iter=4),
        # The cost of one block's parameters without a context (a caller under graph capture, a line search).
        case("cost_block", "cost", nx=20, ny=15, n_pts=60_011),
    ]


def draw(rng):
    """One more case of the same ranges: scenes of 16 to 60,000 cameras and 400 to 6 million points."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(["step", "step", "step", "shared_step", "solve", "retry", "pcg", "pcg", "triangulate", "cost"])
    c = dict(op=op, ring=0, step_x=1.0, nearest=True, n_long=0, n_phys=0, precision="fp64", precond="block_jacobi",
             deflate=False, solver_fp32=False, lam=rng.choice([1e-4, 1e-3]), tol=1e-6, max_iter=4)
    cams = log_int(16, 60_000 if op == "pcg" else 15_000)
    if op == "shared_step":
        cams = log_int(16, 1_000)
    shape = rng.choice(["block", "block", "partition", "strips"]) if cams >= 64 else "block"
    if shape == "strips":
        c.update(ny=5, nx=max(13, cams // 5), step_x=0.5)
    else:
        c.update(nx=max(4, int(math.sqrt(cams * rng.uniform(0.6, 1.6)))))
        c.update(ny=max(4, cams // c["nx"]))
        if shape == "partition" and op != "shared_step":
            c.update(ring=2, nearest=False)
    per_cam = log_int(30, 400)
    n_cams = c["nx"] * c["ny"]
    c["n_pts"] = min(max(400, n_cams * per_cam + rng.randrange(97)), 3_000_000 if op == "pcg" else 6_000_000)
    if op == "shared_step":
        c.update(n_phys=rng.randint(1, 5), lam=1e-2, tol=1e-10, max_iter=1000)
    elif op in ("step", "solve", "retry", "pcg"):
        c["precision"] = rng.choice(["fp64", "fp64", "mixed"])
        c["solver_fp32"] = rng.random() < 0.25
        if n_cams > 4000:
            c["max_iter"] = rng.randint(8, 64 if op == "pcg" else 32)
        else:
            c.update(precond=rng.choice(["block_jacobi", "block_jacobi", "fsai"]), lam=1e-2, tol=1e-12, max_iter=1000)
            c["deflate"] = c["precond"] == "fsai" and rng.random() < 0.5
            if n_cams >= 150 and shape == "block" and rng.random() < 0.3:
                c["n_long"] = rng.randint(1, 6)
    return c


# ---------------------------------------------------------------------------
# scenes (torch, on the GPU)
# ---------------------------------------------------------------------------

class Scene:
    """Inputs of a case: parameters [n_cams][9] (or exterior and interior parts), points, observations."""


def _rotation(w):
    """R and the right Jacobian of the axis-angle map, [n][3][3] each (angles away from 0)."""
    th = w.norm(dim=1)[:, None, None]
    K = torch.zeros(w.shape[0], 3, 3, dtype=F64, device=w.device)
    K[:, 0, 1], K[:, 0, 2] = -w[:, 2], w[:, 1]
    K[:, 1, 0], K[:, 1, 2] = w[:, 2], -w[:, 0]
    K[:, 2, 0], K[:, 2, 1] = -w[:, 1], w[:, 0]
    K2 = K @ K
    eye = torch.eye(3, dtype=F64, device=w.device)
    omc = 2 * torch.sin(th / 2) ** 2
    R = eye + torch.sin(th) / th * K + omc / th ** 2 * K2
    Jr = eye - omc / th ** 2 * K + (th - torch.sin(th)) / th ** 3 * K2
    return R, Jr


def _rotvec(R):
    """Axis-angle of rotations by about half a turn around x (nadir cameras)."""
    # unit quaternion with the x component the largest
    qx = 0.5 * torch.sqrt(1 + R[:, 0, 0] - R[:, 1, 1] - R[:, 2, 2])
    q = torch.stack([qx, (R[:, 0, 1] + R[:, 1, 0]) / (4 * qx), (R[:, 0, 2] + R[:, 2, 0]) / (4 * qx)], 1)
    qw = (R[:, 2, 1] - R[:, 1, 2]) / (4 * qx)
    n = q.norm(dim=1)
    return q * (2 * torch.atan2(n, qw) / n)[:, None]


def _nearest_cams(xs, ys, pts, t, pool, nearest, gen, cam_id):
    """Observations (point, camera), sorted: of each point its t nearest grid cameras, or t of its pool nearest."""
    nx, ny = len(xs), len(ys)
    kx, ky = min(nx, 13 if nx > 3 * ny else 7), min(ny, 7)
    dx, dy = float(xs[1] - xs[0]), float(ys[1] - ys[0])
    op, oc = [], []
    chunk = 1 << 20
    for s in range(0, pts.shape[0], chunk):
        P = pts[s:s + chunk]
        n = P.shape[0]
        ix = ((P[:, 0] - xs[0]) / dx).round().long() - kx // 2
        iy = ((P[:, 1] - ys[0]) / dy).round().long() - ky // 2
        ix, iy = ix.clamp(0, nx - kx), iy.clamp(0, ny - ky)
        gx = (ix[:, None] + torch.arange(kx, device=DEV)).repeat_interleave(ky, 1)
        gy = (iy[:, None] + torch.arange(ky, device=DEV)).repeat(1, kx)
        d = (xs[gx] - P[:, 0:1]) ** 2 + (ys[gy] - P[:, 1:2]) ** 2
        k = min(pool, kx * ky)
        idx = torch.topk(d, k, dim=1, largest=False).indices
        cams = cam_id[gy.gather(1, idx) * nx + gx.gather(1, idx)]
        if not nearest:
            order = torch.rand(cams.shape, generator=gen, device=DEV).argsort(1)
            cams = cams.gather(1, order)
        keep = torch.arange(k, device=DEV)[None, :] < t[s:s + n, None]
        cams = torch.where(keep, cams, 1 << 30).sort(1).values
        keep = cams < (1 << 30)
        op.append((torch.arange(s, s + n, device=DEV)[:, None].expand(n, k))[keep])
        oc.append(cams[keep])
    return torch.cat(op), torch.cat(oc)


def make_scene(c, seed):
    """The case's scene: nadir cameras on a grid, starting parameters a little off, pixels with N(0, 0.5) noise."""
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 17)

    def uni(n, lo, hi):
        return torch.rand(n, generator=g, device=DEV, dtype=F64) * (hi - lo) + lo

    def gauss(*shape):
        return torch.randn(*shape, generator=g, device=DEV, dtype=F64)

    s = Scene()
    nx, ny, ring = c["nx"], c["ny"], c["ring"]
    tiny = nx * ny <= 16
    sx, sy, alt, relief = (2.5, 2.5, 10.0, 1.0) if tiny else (c["step_x"], 1.0, 2.5, 0.25)
    xs = torch.arange(-ring, nx + ring, device=DEV, dtype=F64) * sx
    ys = torch.arange(-ring, ny + ring, device=DEV, dtype=F64) * sy
    gx, gy = xs.repeat(len(ys)), ys.repeat_interleave(len(xs))
    free = (gx >= 0) & (gx < (nx - 0.5) * sx) & (gy >= 0) & (gy < (ny - 0.5) * sy)
    order = torch.cat([free.nonzero()[:, 0], (~free).nonzero()[:, 0]])   # free cameras first
    cam_id = torch.empty_like(order)
    cam_id[order] = torch.arange(len(order), device=DEV)
    gx, gy, free = gx[order], gy[order], free[order]
    s.n_cams = len(order)
    s.fixed = (~free).to(torch.uint8) if ring else None
    centres = torch.stack([gx, gy, torch.full_like(gx, alt)], 1)
    # points over the covered ground, and a few distant ones that many cameras see
    half = 0.0 if tiny else (0.5 if ring else 0.5 * alt)
    n_near = c["n_pts"] - c["n_long"]
    pts = torch.stack([uni(n_near, -half, (nx - 1) * sx + half), uni(n_near, -half, (ny - 1) * sy + half),
                       uni(n_near, 0.0, relief)], 1)
    if tiny:
        t = torch.randint(2, 7, (n_near,), generator=g, device=DEV)
    else:
        w = Q_TRACK ** torch.arange(11, device=DEV, dtype=F64)
        cdf = (w / w.sum()).cumsum(0)
        t = 2 + torch.searchsorted(cdf, uni(n_near, 0.0, 1.0)).clamp(max=10)
    pool = 16 if tiny else 12
    obs_pt, obs_cam = _nearest_cams(xs, ys, pts, t, pool, c["nearest"] and not tiny, g, cam_id)
    if c["n_long"]:
        n = c["n_long"]
        far = torch.stack([uni(n, 0.4, 0.6) * float(xs[-1]), uni(n, 0.4, 0.6) * float(ys[-1]),
                           torch.full((n,), -20.0, dtype=F64, device=DEV)], 1)
        most = min(s.n_cams, 300)
        for j in range(n):
            seen = LONG_FROM + (j * (most - LONG_FROM)) // max(1, n - 1 if n > 1 else 1)
            d = (centres[:, 0] - far[j, 0]) ** 2 + (centres[:, 1] - far[j, 1]) ** 2
            cams = torch.topk(d, min(seen, s.n_cams), largest=False).indices.sort().values
            obs_pt = torch.cat([obs_pt, torch.full_like(cams, n_near + j)])
            obs_cam = torch.cat([obs_cam, cams])
        pts = torch.cat([pts, far])
    s.n_pts, s.n_obs = pts.shape[0], obs_pt.shape[0]
    # attitude: half a turn about x with a small tilt; t = -R C
    tilt, _ = _rotation(gauss(s.n_cams, 3) * 0.02)
    nadir = torch.tensor([[1.0, 0, 0], [0, -1, 0], [0, 0, -1]], dtype=F64, device=DEV)
    R = tilt @ nadir
    n_phys = c["n_phys"]
    n_int = n_phys or s.n_cams
    f, k1, k2 = uni(n_int, 950, 1050), uni(n_int, -0.05, 0.05), uni(n_int, -0.01, 0.01)
    pp = uni((2 * n_int) if n_phys else 0, -5, 5).reshape(2, -1)

    def exterior(R, C):
        return torch.cat([_rotvec(R), -(R @ C[:, :, None])[:, :, 0]], 1)

    turn, _ = _rotation(gauss(s.n_cams, 3) * 0.002)
    moved = centres + gauss(s.n_cams, 3) * 0.01
    start = exterior(turn @ R, moved)
    true = exterior(R, centres)
    if s.fixed is not None:
        start[~free] = true[~free]
    s.pts0 = pts + gauss(*pts.shape) * 0.01
    s.obs_pt, s.obs_cam = obs_pt, obs_cam
    if n_phys:
        s.img_cam = torch.arange(s.n_cams, device=DEV) % n_phys
        intr = torch.stack([f, pp[0], pp[1], k1, k2], 1)
        s.ext0, s.int0 = start, intr
        uv = project(true, intr, s.img_cam, pts, obs_cam, obs_pt)[0]
    else:
        s.img_cam = None
        intr = torch.stack([f, torch.zeros_like(f), torch.zeros_like(f), k1, k2], 1)
        s.ext0, s.int0 = start, intr
        uv = project(true, intr, None, pts, obs_cam, obs_pt)[0]
        s.cams0 = torch.cat([start, f[:, None], k1[:, None], k2[:, None]], 1).contiguous()
    s.uv = uv + gauss(2, s.n_obs) * 0.5
    s.lm_cams = int(free.sum())
    return s


def project(ext, intr, img_cam, pts, obs_cam, obs_pt, jac=False):
    """Pixels [2][n] of all observations, and with jac the derivatives by the exterior (6), the interior (5: f, cx,
    cy, k1, k2) and the point (3), [n][2][.] each."""
    R, Jr = _rotation(ext[:, 0:3])
    X = pts[obs_pt]
    Ro = R[obs_cam]
    RX = (Ro @ X[:, :, None])[:, :, 0]
    P = RX + ext[obs_cam, 3:6]
    q = intr[img_cam[obs_cam]] if img_cam is not None else intr[obs_cam]
    iz = 1 / P[:, 2]
    x, y = P[:, 0] * iz, P[:, 1] * iz
    r2 = x * x + y * y
    f, k1, k2 = q[:, 0], q[:, 3], q[:, 4]
    d = 1 + k1 * r2 + k2 * r2 * r2
    uv = torch.stack([f * d * x + q[:, 1], f * d * y + q[:, 2]])
    if not jac:
        return uv, None, None, None
    n = len(x)
    dd = 2 * (k1 + 2 * k2 * r2)
    A = torch.empty(n, 2, 2, dtype=F64, device=pts.device)
    A[:, 0, 0], A[:, 1, 1] = f * (d + x * x * dd), f * (d + y * y * dd)
    A[:, 0, 1] = A[:, 1, 0] = f * x * y * dd
    B = torch.zeros(n, 2, 3, dtype=F64, device=pts.device)
    B[:, 0, 0] = B[:, 1, 1] = iz
    B[:, 0, 2], B[:, 1, 2] = -x * iz, -y * iz
    E = A @ B                                        # d pixel / d P
    # dP/dw = -R [X]x J_r(w), with R [X]x = [R X]x R
    S = torch.zeros(n, 3, 3, dtype=F64, device=pts.device)
    S[:, 0, 1], S[:, 0, 2], S[:, 1, 2] = -RX[:, 2], RX[:, 1], -RX[:, 0]
    S -= S.transpose(1, 2).clone()
    Jw = -(E @ (S @ (Ro @ Jr[obs_cam])))
    Je = torch.cat([Jw, E], 2)
    Ji = torch.zeros(n, 2, 5, dtype=F64, device=pts.device)
    Ji[:, 0, 0], Ji[:, 1, 0] = d * x, d * y
    Ji[:, 0, 1] = Ji[:, 1, 2] = 1
    Ji[:, 0, 3], Ji[:, 1, 3] = f * x * r2, f * y * r2
    Ji[:, 0, 4], Ji[:, 1, 4] = f * x * r2 * r2, f * y * r2 * r2
    return uv, Je, Ji, E @ Ro


# ---------------------------------------------------------------------------
# the passes
# ---------------------------------------------------------------------------

PRECOND = {"block_jacobi": ba.BA_PRECOND_BLOCK_JACOBI, "fsai": ba.BA_PRECOND_FSAI,
           "learned_fsai": ba.BA_PRECOND_LEARNED_FSAI}


class State:
    """A program's context with its parameters and result arrays."""
    ctx = net = None

    def __del__(self):
        if self.ctx:
            ba.ba_destroy(self.ctx)
        if self.net:
            ba.ba_gnn_destroy(self.net)


def prepare(case, seed):
    s = make_scene(case, seed)
    st = State()
    st.case = case
    st.obs = (s.obs_cam.to(torch.int32), s.obs_pt.to(torch.int32), s.uv)
    st.pts0 = s.pts0
    if case["op"] == "cost":
        st.cams0 = s.cams0
        st.cost = torch.zeros(1, dtype=F64, device=DEV)
        return st
    if case["op"] == "shared_step":
        st.cams0 = torch.cat([s.ext0.reshape(-1), s.int0.reshape(-1)]).contiguous()
        st.ctx = ba.ba_create_shared(s.n_cams, case["n_phys"], s.n_pts, *st.obs, s.img_cam.to(torch.int32))
    else:
        st.cams0 = s.cams0
        st.ctx = ba.ba_create(s.n_cams, s.n_pts, *st.obs, cam_fixed=s.fixed,
                              precision=ba.BA_MIXED if case["precision"] == "mixed" else ba.BA_FP64)
    st.obs = None                      # the context has its own copy
    st.opts = dict(precond=PRECOND[case["precond"]], deflate=case["deflate"], solver_fp32=case["solver_fp32"])
    if case["precond"] == "learned_fsai":
        weights = np.load(ba._HERE + "/learned_precond_fsai_weights.npy", allow_pickle=False)
        st.net = ba.ba_gnn_create(weights, stream=torch.cuda.current_stream())
        ba.ba_set_preconditioner_net(st.ctx, st.net)
    n_rows = ba.ba_get_sizes(st.ctx)["n_rows"]
    st.dxc = torch.zeros(n_rows, 9, dtype=F64, device=DEV)
    st.dxp = torch.zeros(s.n_pts, 3, dtype=F64, device=DEV)
    if case["op"] in ("retry", "pcg"):
        ba.ba_linearize(st.ctx, st.cams0, st.pts0)
    if case["op"] == "pcg":
        ba.ba_form_rcs(st.ctx, case["lam"])
    return st


def run(st):
    c = st.case
    op = c["op"]
    if op in ("step", "shared_step"):
        # the caller keeps its parameters until the step is known to be good
        cams, pts = st.cams0.clone(), st.pts0.clone()
        info = ba.ba_lm_step(st.ctx, cams, pts, ba.new_lm_state(c["lam"]), pcg_tol=c["tol"],
                             pcg_max_iter=c["max_iter"], **st.opts)
        return dict(cams=cams, pts=pts, cost=info["cost"], cost_new=info["cost_new"], accepted=info["accepted"])
    if op == "triangulate":
        pts = st.pts0.clone()
        failed = ba.ba_triangulate(st.ctx, st.cams0, pts, linear_init=True, n_gn=c["max_iter"])
        return dict(pts=pts, failed=failed)
    if op == "cost":
        ba.ba_cost_noalloc(st.cams0, st.pts0, *st.obs, st.cost)
        return dict(cost=st.cost)
    out = {}
    if op == "solve":
        out["cost"] = ba.ba_linearize(st.ctx, st.cams0, st.pts0)
    if op != "pcg":
        ba.ba_form_rcs(st.ctx, c["lam"])
    ba.ba_pcg_solve(st.ctx, st.dxc, tol=c["tol"], max_iter=c["max_iter"], **st.opts)
    out["dxc"] = st.dxc
    if op != "pcg":
        ba.ba_back_substitute(st.ctx, st.dxc, st.dxp)
        out["dxp"] = st.dxp
    return out


def work(case):
    """Least bytes and operations of a pass: observations (8 + 16 bytes) and parameters once, results once; a solve
    reads the stored upper blocks of S (about 10 + 0.5 x the 30 neighbours a row) once an iteration."""
    c = case
    n_pts, rows = c["n_pts"], c["nx"] * c["ny"]
    n_obs = 4.0 * n_pts + 150 * c["n_long"]
    params = 72.0 * rows + 24.0 * n_pts
    if c["op"] == "cost":
        return {"bytes": 24 * n_obs + params, "flops": 110 * n_obs}
    if c["op"] == "triangulate":
        return {"bytes": 24 * n_obs + params + 24 * n_pts, "flops": n_obs * (300 + 250 * c["max_iter"])}
    blocks = rows * min(24.0, (rows + 1) / 2)
    iters = min(c["max_iter"], 60 if c["precond"] == "block_jacobi" else 30)   # about what the tolerances need
    size = 4 if c["solver_fp32"] else 8
    pcg_bytes = iters * (81.0 * size * blocks + 72 * 6 * rows) + 72 * rows
    pcg_flops = iters * (4 * 81.0 * blocks + 300 * rows)
    if c["precond"] != "block_jacobi":
        pcg_bytes += iters * 81 * 4 * blocks
        pcg_flops += iters * 4 * 81.0 * blocks + rows * (9.0 * 28) ** 3 / 3
    if c["op"] == "pcg":
        return {"bytes": pcg_bytes, "flops": pcg_flops}
    pairs = 2.1 * n_obs
    form_flops = 400 * pairs + 700 * n_obs
    return {"bytes": 24 * n_obs + 2 * params + 648 * blocks + pcg_bytes, "flops": form_flops + pcg_flops}


# ---------------------------------------------------------------------------
# the same results in 64 bits from the definitions, plain torch
# ---------------------------------------------------------------------------

def _chol3(V):
    """Lower Cholesky factors of [n][3][3]."""
    L = torch.zeros_like(V)
    L[:, 0, 0] = V[:, 0, 0].sqrt()
    L[:, 1, 0], L[:, 2, 0] = V[:, 1, 0] / L[:, 0, 0], V[:, 2, 0] / L[:, 0, 0]
    L[:, 1, 1] = (V[:, 1, 1] - L[:, 1, 0] ** 2).sqrt()
    L[:, 2, 1] = (V[:, 2, 1] - L[:, 2, 0] * L[:, 1, 0]) / L[:, 1, 1]
    L[:, 2, 2] = (V[:, 2, 2] - L[:, 2, 0] ** 2 - L[:, 2, 1] ** 2).sqrt()
    return L


def _solve3(A, b):
    """x = A^-1 b for SPD [n][3][3] by Cholesky."""
    L = _chol3(A)
    y0 = b[:, 0] / L[:, 0, 0]
    y1 = (b[:, 1] - L[:, 1, 0] * y0) / L[:, 1, 1]
    y2 = (b[:, 2] - L[:, 2, 0] * y0 - L[:, 2, 1] * y1) / L[:, 2, 2]
    x2 = y2 / L[:, 2, 2]
    x1 = (y1 - L[:, 2, 1] * x2) / L[:, 1, 1]
    x0 = (y0 - L[:, 1, 0] * x1 - L[:, 2, 0] * x2) / L[:, 0, 0]
    return torch.stack([x0, x1, x2], 1)


def _by_point(n_pts, obs_pt, v):
    return torch.zeros(n_pts, *v.shape[1:], dtype=F64, device=v.device).index_add_(0, obs_pt, v)


class Normal:
    """Damped normal equations with the points eliminated: S v, its right-hand side and diagonal blocks, without
    forming S.  Unknowns: `groups` of (row of each observation or -1, J [n][2][k], number of rows)."""

    def __init__(self, groups, Jp, e, obs_pt, n_pts, lam):
        self.groups, self.obs_pt, self.n_pts, self.Jp = groups, obs_pt, n_pts, Jp
        JpT = Jp.transpose(1, 2)
        V = _by_point(n_pts, obs_pt, JpT @ Jp)
        V = V + lam * torch.diag_embed(torch.diagonal(V, dim1=1, dim2=2))
        self.Vinv = torch.linalg.inv(V)
        self.lp = _by_point(n_pts, obs_pt, -(JpT @ e[:, :, None])[:, :, 0])
        self.diagU, self.rhs = [], []
        e2 = e + (Jp @ (self.Vinv @ self.lp[:, :, None])[obs_pt])[:, :, 0]
        for row, J, n in groups:
            keep = row >= 0
            U = torch.zeros(n, J.shape[2], dtype=F64, device=J.device)
            U.index_add_(0, row[keep], (J * J).sum(1)[keep])
            b = torch.zeros(n, J.shape[2], dtype=F64, device=J.device)
            b.index_add_(0, row[keep], -(J.transpose(1, 2) @ e2[:, :, None])[:, :, 0][keep])
            self.diagU.append(lam * U)
            self.rhs.append(b)

    def jx(self, xs):
        """J_c x per observation."""
        y = 0
        for (row, J, n), x in zip(self.groups, xs):
            v = (J @ x[row.clamp(min=0)][:, :, None])[:, :, 0]
            y = y + torch.where((row >= 0)[:, None], v, 0.0)
        return y

    def points(self, xs):
        """Eq. (5): the points' part for given camera parts."""
        w = _by_point(self.n_pts, self.obs_pt, (self.Jp.transpose(1, 2) @ self.jx(xs)[:, :, None])[:, :, 0])
        return (self.Vinv @ (self.lp - w)[:, :, None])[:, :, 0]

    def product(self, xs):
        y = self.jx(xs)
        w = _by_point(self.n_pts, self.obs_pt, (self.Jp.transpose(1, 2) @ y[:, :, None])[:, :, 0])
        y = y - (self.Jp @ (self.Vinv @ w[:, :, None])[self.obs_pt])[:, :, 0]
        out = []
        for (row, J, n), x, lu in zip(self.groups, xs, self.diagU):
            keep = row >= 0
            out.append((lu * x).index_add_(0, row[keep], (J.transpose(1, 2) @ y[:, :, None])[:, :, 0][keep]))
        return out

    def diagonal_inverses(self):
        out = []
        for (row, J, n), lu in zip(self.groups, self.diagU):
            k = J.shape[2]
            D = torch.zeros(n, k, k, dtype=F64, device=J.device)
            step = 1 << 21
            for a in range(0, len(row), step):
                r, j = row[a:a + step], J[a:a + step]
                keep = r >= 0
                D.index_add_(0, r[keep], (j.transpose(1, 2) @ j)[keep])
                if n == int(row.max()) + 1 and k == 5:   # few physical cameras: below, over all their images
                    continue
                jp = self.Jp[a:a + step]
                W = j.transpose(1, 2) @ jp
                D.index_add_(0, r[keep], -(W @ self.Vinv[self.obs_pt[a:a + step]] @ W.transpose(1, 2))[keep])
            if k == 5:
                W = J.transpose(1, 2) @ self.Jp
                for c in range(n):
                    on = row == c
                    T = _by_point(self.n_pts, self.obs_pt[on], W[on])
                    D[c] -= (T @ self.Vinv @ T.transpose(1, 2)).sum(0)
            D = D + torch.diag_embed(lu)
            out.append(torch.linalg.inv(0.5 * (D + D.transpose(1, 2))))
        return out


def _dot(a, b):
    return sum(float((x * y).sum()) for x, y in zip(a, b))


def _pcg(N, tol, max_iter):
    M = N.diagonal_inverses()

    def prec(r):
        return [(m @ v[:, :, None])[:, :, 0] for m, v in zip(M, r)]

    x = [torch.zeros_like(b) for b in N.rhs]
    r = [b.clone() for b in N.rhs]
    z = prec(r)
    d = [v.clone() for v in z]
    rz, r0 = _dot(r, z), math.sqrt(_dot(r, r))
    for _ in range(max_iter):
        if math.sqrt(_dot(r, r)) <= tol * r0:
            break
        q = N.product(d)
        alpha = rz / _dot(d, q)
        x = [a + alpha * b for a, b in zip(x, d)]
        r = [a - alpha * b for a, b in zip(r, q)]
        z = prec(r)
        rz, old = _dot(r, z), rz
        d = [a + rz / old * b for a, b in zip(z, d)]
    return x


def _exact_triangulate(c, s):
    """Linear start and Gauss-Newton steps of every point."""
    ext, intr, n_pts, op, oc = s.ext0, s.int0, s.n_pts, s.obs_pt, s.obs_cam
    R, _ = _rotation(ext[:, :3])
    q, t, Ro = intr[oc], ext[oc, 3:6], R[oc]
    rho = (s.uv[0] ** 2 + s.uv[1] ** 2).sqrt() / q[:, 0]
    r = rho.clone()
    for _ in range(30):
        r2 = r * r
        r = r - (r * (1 + q[:, 3] * r2 + q[:, 4] * r2 * r2) - rho) / (1 + 3 * q[:, 3] * r2 + 5 * q[:, 4] * r2 * r2)
    scale = torch.where(rho > 0, r / rho, torch.ones_like(rho)) / q[:, 0]
    xy = s.uv * scale
    A = xy.T[:, :, None] * Ro[:, 2:3, :] - Ro[:, 0:2, :]
    b = t[:, 0:2] - xy.T * t[:, 2:3]
    AT = A.transpose(1, 2)
    X = _solve3(_by_point(n_pts, op, AT @ A), _by_point(n_pts, op, (AT @ b[:, :, None])[:, :, 0]))
    for _ in range(c["max_iter"]):
        uv, _, _, Jp = project(ext, intr, None, X, oc, op, jac=True)
        JT = Jp.transpose(1, 2)
        e = (uv - s.uv).T
        X = X + _solve3(_by_point(n_pts, op, JT @ Jp), _by_point(n_pts, op, -(JT @ e[:, :, None])[:, :, 0]))
    return X


def exact(case, seed):
    c, op = case, case["op"]
    s = make_scene(c, seed)
    if op == "triangulate":
        return dict(pts=_exact_triangulate(c, s), failed=None)
    uv, Je, Ji, Jp = project(s.ext0, s.int0, s.img_cam, s.pts0, s.obs_cam, s.obs_pt, jac=op != "cost")
    e = (uv - s.uv).T.contiguous()
    cost = 0.5 * (e * e).sum()
    if op == "cost":
        return dict(cost=cost.reshape(1))
    n_cams = s.n_cams
    if s.img_cam is not None:
        groups = [(s.obs_cam, Je, n_cams), (s.img_cam[s.obs_cam], Ji, c["n_phys"])]
    else:
        row = s.obs_cam if s.fixed is None else torch.where(s.fixed[s.obs_cam] > 0, -1, s.obs_cam)
        groups = [(row, torch.cat([Je, Ji[:, :, [0, 3, 4]]], 2), s.lm_cams)]
    del Je, Ji
    N = Normal(groups, Jp, e, s.obs_pt, s.n_pts, c["lam"])
    if c["precond"] == "block_jacobi":
        x = _pcg(N, c["tol"], c["max_iter"])
    else:
        x = _pcg(N, 1e-14, 1500)           # the solution: these cases solve to a tight tolerance
    if op == "pcg":
        return dict(dxc=x[0])
    dxp = N.points(x)
    if op in ("solve", "retry"):
        out = dict(dxc=x[0], dxp=dxp)
        if op == "solve":
            out["cost"] = cost
        return out
    ext, intr = s.ext0.clone(), s.int0.clone()
    if s.img_cam is not None:
        ext += x[0]
        intr += x[1]
        cams = torch.cat([ext.reshape(-1), intr.reshape(-1)])
    else:
        ext[:s.lm_cams] += x[0][:, :6]
        intr[:s.lm_cams][:, [0, 3, 4]] += x[0][:, 6:]
        intr[:s.lm_cams] = torch.cat([(s.int0[:s.lm_cams, 0:1] + x[0][:, 6:7]), s.int0[:s.lm_cams, 1:3],
                                      s.int0[:s.lm_cams, 3:5] + x[0][:, 7:9]], 1)
        cams = torch.cat([ext, intr[:, [0, 3, 4]]], 1)
    pts = s.pts0 + dxp
    e = (project(ext, intr, s.img_cam, pts, s.obs_cam, s.obs_pt)[0] - s.uv).T
    cost_new = 0.5 * (e * e).sum()
    if not bool(cost_new < cost):          # a rejected step leaves the parameters
        cams = torch.cat([s.ext0.reshape(-1), s.int0.reshape(-1)]) if s.img_cam is not None else s.cams0
        pts = s.pts0
    return dict(cams=cams, pts=pts, cost=cost, cost_new=cost_new, accepted=None)
