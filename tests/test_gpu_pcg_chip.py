"""The PCG solve that runs in one kernel with S in registers (systems whose
rows fit the chip, FULL layout) against the kernels that a larger system or
the UPPER layout takes (needs a GPU): one workgroup and many, every number of
blocks a lane group holds, the row limit of a workgroup, dense rows, systems
that do not fit, the stops, an initial guess, repeated and concurrent solves."""
import threading

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2307_08383_amd import scenegen

from gpu_util import T, create

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ba = pytest.importorskip("paper_2307_08383_amd.ba")

LAM = 1e-2


def _grid(nx, ny, n_pts):
    return lambda: scenegen.aerial_grid_scene(seed=3, nx=nx, ny=ny, n_pts=n_pts, with_stats=False)


def _fixed_but_one():
    s = scenegen.aerial_grid_scene(seed=3, nx=4, ny=3, n_pts=300, with_stats=False)
    s.cam_fixed[1:] = 1
    return s


SCENES = {
    "one row": _fixed_but_one,                       # a 9x9 system
    "tiny": lambda: scenegen.tiny_scene(seed=0, with_stats=False),   # one workgroup
    "30 rows": _grid(6, 5, 3000),                    # one workgroup or few
    "40 rows in line": _grid(40, 1, 2000),           # the row limit of a workgroup
    "41 rows in line": _grid(41, 1, 2000),
    "80 rows": _grid(10, 8, 12000),
    "300 rows": _grid(20, 15, 40000),
    "750 rows": _grid(30, 25, 90000),
    "1369 rows": _grid(37, 37, 150000),
    "2000 rows": _grid(50, 40, 200000),              # most of the registers
    "4096 rows": _grid(64, 64, 300000),              # does not fit: one kernel per phase
    "dense": lambda: scenegen.long_track_scene(n_pts=4000, long_tracks=(65, 200, 300)),   # rows of up to 300 blocks
}


def _formed(scene, stream=None):
    uv = orc.observations(scene)
    ctx = create(scene, uv, 0)
    ba.ba_linearize(ctx, T(scene.cams_init, torch.float64), T(scene.pts_init, torch.float64))
    ba.ba_form_rcs(ctx, LAM)
    return ctx


def _solve(ctx, n_rows, **kw):
    x = torch.full((n_rows, 9), 7.0, dtype=torch.float64, device="cuda")
    info = ba.ba_pcg_solve(ctx, x, **kw)
    return info, x


def _residual(ctx, x, b):
    y = torch.empty_like(x)
    ba.ba_rcs_product(ctx, x, y, product=ba.BA_PRODUCT_UPPER)
    return float((b - y).norm() / b.norm())


# (one camera among fixed ones has no gauge freedom: deflating seven of its
# nine directions leaves nothing to converge, in any layout)
@pytest.mark.parametrize("name,deflate", [(n, d) for n in SCENES for d in (False, True) if not (d and n == "one row")])
@pytest.mark.parametrize("precond", ["block_jacobi", "fsai"])
def test_same_solution_as_the_kernels_per_phase(name, deflate, precond):
    """Both stop at 1e-12: iterations within the margin of different rounding
    (FSAI: of the UPPER layout's FP16 factor too), the true residuals alike,
    and (with the damping of 1e-2, which bounds the Jacobi-scaled system's
    condition by a few thousand) the solutions to 1e-8.  A second solve
    repeats the first bit by bit."""
    ctx = _formed(SCENES[name]())
    pre = ba.BA_PRECOND_FSAI if precond == "fsai" else ba.BA_PRECOND_BLOCK_JACOBI
    try:
        n = ba.ba_get_sizes(ctx)["n_rows"]
        b = T(ba.ba_get_rcs(ctx)[1], torch.float64)
        kw = dict(tol=1e-12, max_iter=3000, precond=pre, deflate=deflate)
        i1, x1 = _solve(ctx, n, **kw)
        i2, x2 = _solve(ctx, n, **kw)
        iu, xu = _solve(ctx, n, product=ba.BA_PRODUCT_UPPER, **kw)
        r1, ru = _residual(ctx, x1, b), _residual(ctx, xu, b)
    finally:
        ba.ba_destroy(ctx)
    assert i1["status"] == i2["status"] == iu["status"] == 0
    assert i1["iters"] == i2["iters"] and torch.equal(x1, x2)
    assert i1["relres"] <= 1e-12
    assert abs(i1["iters"] - iu["iters"]) <= max(5 if precond == "fsai" else 3, 0.1 * iu["iters"])
    assert r1 <= 10 * max(ru, 1e-12), (r1, ru)
    assert float((x1 - xu).norm()) <= 1e-8 * float(xu.norm())


@pytest.mark.parametrize("name", ["tiny", "80 rows", "2000 rows"])
def test_solver_matrix_in_fp32(name):
    """The products with S rounded to FP32: both layouts solve the same
    rounded system."""
    ctx = _formed(SCENES[name]())
    try:
        n = ba.ba_get_sizes(ctx)["n_rows"]
        kw = dict(tol=1e-12, max_iter=3000, solver_fp32=True)
        i1, x1 = _solve(ctx, n, **kw)
        iu, xu = _solve(ctx, n, product=ba.BA_PRODUCT_UPPER, **kw)
        _, x64 = _solve(ctx, n, tol=1e-12, max_iter=3000)
    finally:
        ba.ba_destroy(ctx)
    assert i1["status"] == iu["status"] == 0
    assert float((x1 - xu).norm()) <= 1e-8 * float(xu.norm())
    assert not torch.equal(x1, x64)


@pytest.mark.parametrize("name", ["tiny", "80 rows", "dense"])
def test_stops_and_initial_guess(name):
    """The iteration cap, no iteration at all, a guess that is the solution,
    and a guess on the way to it."""
    ctx = _formed(SCENES[name]())
    try:
        n = ba.ba_get_sizes(ctx)["n_rows"]
        i0, x0 = _solve(ctx, n, tol=1e-12, max_iter=0)
        assert i0["status"] == ba.BA_ERR_NOT_CONVERGED and i0["iters"] == 0 and i0["relres"] == 1.0
        assert float(x0.abs().max()) == 0.0
        i3, x3 = _solve(ctx, n, tol=0.0, max_iter=3)
        u3, y3 = _solve(ctx, n, tol=0.0, max_iter=3, product=ba.BA_PRODUCT_UPPER)
        assert i3["status"] == u3["status"] == ba.BA_ERR_NOT_CONVERGED and i3["iters"] == u3["iters"] == 3
        # three steps of the same recurrence differ by rounding alone
        assert float((x3 - y3).norm()) <= 1e-12 * float(y3.norm())
        assert abs(i3["relres"] - u3["relres"]) <= 1e-12 * u3["relres"]
        ia, xa = _solve(ctx, n, tol=1e-12, max_iter=3000)
        ib, xb = _solve(ctx, n, tol=1e-12, max_iter=3000, x0=x3)
        assert ib["status"] == 0 and float((xa - xb).norm()) <= 1e-7 * float(xa.norm())
        loose, xl = _solve(ctx, n, tol=0.5, max_iter=3000, x0=xa)
        # |r_0| is the guess's: a factor two takes few steps, and the solution stays
        assert loose["iters"] <= 20 and float((xl - xa).norm()) <= 1e-7 * float(xa.norm())
    finally:
        ba.ba_destroy(ctx)


def test_solves_from_two_threads_and_streams():
    """Two contexts on two streams solve at the same time, each as alone."""
    scenes = [SCENES["300 rows"](), SCENES["750 rows"]()]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    ctxs, rows, alone = [], [], []
    for s, st in zip(scenes, streams):
        uv = orc.observations(s)
        with torch.cuda.stream(st):
            ctx = create(s, uv, 0)
            ba.ba_linearize(ctx, T(s.cams_init, torch.float64), T(s.pts_init, torch.float64))
            ba.ba_form_rcs(ctx, LAM)
            ctxs.append(ctx)
            rows.append(ba.ba_get_sizes(ctx)["n_rows"])
            alone.append(_solve(ctx, rows[-1], tol=1e-10, max_iter=3000)[1].cpu())
    got = [[], []]

    def work(i):
        with torch.cuda.stream(streams[i]):
            for _ in range(10):
                got[i].append(_solve(ctxs[i], rows[i], tol=1e-10, max_iter=3000)[1].cpu())

    th = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    for ctx in ctxs:
        ba.ba_destroy(ctx)
    for i in range(2):
        assert len(got[i]) == 10
        for x in got[i]:
            assert torch.equal(x, alone[i])
