"""Rounding of the Gauss-Newton re-triangulation far from the origin (needs a
GPU): points hundreds of units from it, against extended precision on the
same inputs."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2307_08383_amd import scenegen

from gpu_util import T, create

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ba = pytest.importorskip("paper_2307_08383_amd.ba")


def gauss_newton(s, uv, n, dtype):
    """n Gauss-Newton steps of every point from pts_init in `dtype`, the point
    turned by X + a w x X + b w x (w x X)."""
    c = s.cams_init.astype(dtype)[s.obs_cam]
    X = s.pts_init.astype(dtype)
    w = [c[:, i] for i in range(3)]
    s2 = w[0] * w[0] + w[1] * w[1] + w[2] * w[2]
    th = np.sqrt(s2)
    a, b = np.sin(th) / th, 2 * np.sin(th / 2) ** 2 / s2
    f, k1, k2 = c[:, 6], c[:, 7], c[:, 8]

    def cross(v):
        return [w[1] * v[2] - w[2] * v[1], w[2] * v[0] - w[0] * v[2], w[0] * v[1] - w[1] * v[0]]

    for _ in range(n):
        x = [X[s.obs_pt, i] for i in range(3)]
        cx = cross(x)
        cc = cross(cx)
        P = [x[i] + a * cx[i] + b * cc[i] + c[:, 3 + i] for i in range(3)]
        px, py = P[0] / P[2], P[1] / P[2]
        r2 = px * px + py * py
        d, dd = 1 + r2 * (k1 + k2 * r2), k1 + 2 * k2 * r2
        e = [f * d * px - uv[0].astype(dtype), f * d * py - uv[1].astype(dtype)]
        A00, A01, A11 = f * (d + 2 * px * px * dd), f * 2 * px * py * dd, f * (d + 2 * py * py * dd)
        E = [[A00 / P[2], A01 / P[2], -(A00 * px + A01 * py) / P[2]], [A01 / P[2], A11 / P[2], -(A01 * px + A11 * py) / P[2]]]
        R = [[(a * 0 + 1 if i == j else a * 0) + b * (w[i] * w[j] - (s2 if i == j else 0)) for j in range(3)] for i in range(3)]
        for i, j, k, sg in ((0, 1, 2, -1), (0, 2, 1, 1), (1, 0, 2, 1), (1, 2, 0, -1), (2, 0, 1, -1), (2, 1, 0, 1)):
            R[i][j] = R[i][j] + sg * a * w[k]
        J = [[E[r][0] * R[0][j] + E[r][1] * R[1][j] + E[r][2] * R[2][j] for j in range(3)] for r in range(2)]
        A, g = np.zeros((s.n_pts, 3, 3), dtype), np.zeros((s.n_pts, 3), dtype)
        for i in range(3):
            np.add.at(g[:, i], s.obs_pt, -(J[0][i] * e[0] + J[1][i] * e[1]))
            for j in range(3):
                np.add.at(A[:, i, j], s.obs_pt, J[0][i] * J[0][j] + J[1][i] * J[1][j])
        adj = np.stack([np.cross(A[:, 1], A[:, 2]), np.cross(A[:, 2], A[:, 0]), np.cross(A[:, 0], A[:, 1])], 2)
        det = (A[:, 0] * adj[:, :, 0]).sum(1)
        X = X + (adj * g[:, None, :]).sum(2) / det[:, None]
    return X


@pytest.mark.parametrize("nx,ny", [(900, 3), (60, 50)])
def test_error_far_from_the_origin(nx, ny):
    """The library's error is that of the same formula in FP64 numpy but for
    the contraction of products and sums: the median over the points of the
    largest component's error within 1.5 times numpy's.  (Turned by R X, which
    rounds at the size of X, it would be 2 to 3 times as large in the line of
    cameras.)"""
    s = scenegen.aerial_grid_scene(seed=21, nx=nx, ny=ny, n_pts=12_000, with_stats=False)
    uv = orc.observations(s)
    near = np.ones(s.n_pts, bool)   # points of a narrow view, whose steps converge
    np.logical_and.at(near, s.obs_pt, np.linalg.norm(uv, axis=0) / s.cams_init[s.obs_cam, 6] < 1.0)
    exact = gauss_newton(s, uv, 9, np.longdouble)
    numpy64 = gauss_newton(s, uv, 7, np.float64)
    ctx = create(s, uv)
    try:
        pts = T(s.pts_init, torch.float64)
        assert ba.ba_triangulate(ctx, T(s.cams_init, torch.float64), pts, linear_init=False, n_gn=7) == 0
    finally:
        ba.ba_destroy(ctx)

    def median(X):
        return float(np.median(np.abs(X[near] - exact[near]).max(1)))
    assert near.mean() > 0.8
    print("median error", median(pts.cpu().numpy()), "numpy", median(numpy64))
    assert median(pts.cpu().numpy()) <= 1.5 * median(numpy64)
