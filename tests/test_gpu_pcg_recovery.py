"""The PCG solves in one kernel against the kernels that run one phase each
(needs a GPU): a solve that could not be launched, or one of whose workgroups
gave up waiting, is repeated with those as if it had not been tried, and the
solve that keeps their order of sums gives their result bit for bit.
BA_CHIP_GIVE_UP, read at creation: 1 takes the launch as refused, 2 takes one
workgroup to have given up when all have written their results.  Either way
the kernels end normally, and the context solves with one kernel per phase
afterwards, which is the reference here."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2307_08383_amd import scenegen

import test_gpu_pcg_ordered as ordered
from gpu_util import T, create

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ba = pytest.importorskip("paper_2307_08383_amd.ba")

SCENES = {
    "tiny": lambda: scenegen.tiny_scene(seed=0, with_stats=False),   # one workgroup
    "300": lambda: scenegen.aerial_grid_scene(seed=3, nx=20, ny=15, n_pts=40000, with_stats=False),
    "dense": lambda: scenegen.long_track_scene(n_pts=4000, long_tracks=(65, 200, 300)),
}
FORMS = {
    "tight": dict(tol=1e-10), "loose": dict(tol=1e-6), "fp32": dict(tol=1e-10, solver_fp32=True),
    "deflated": dict(tol=1e-10, deflate=True), "fsai": dict(tol=1e-10, precond=ba.BA_PRECOND_FSAI),
    "fsai deflated": dict(tol=1e-10, precond=ba.BA_PRECOND_FSAI, deflate=True),
}


def _context(monkeypatch, scene, give_up=None):
    if give_up is None:
        monkeypatch.delenv("BA_CHIP_GIVE_UP", raising=False)
    else:
        monkeypatch.setenv("BA_CHIP_GIVE_UP", str(give_up))
    return create(scene, orc.observations(scene), 0)


def _form(ctx, s, lam=1e-2):
    ba.ba_linearize(ctx, T(s.cams_init, torch.float64), T(s.pts_init, torch.float64))
    ba.ba_form_rcs(ctx, lam)
    return ba.ba_get_sizes(ctx)["n_rows"]


def _solve(ctx, x, **kw):
    i = ba.ba_pcg_solve(ctx, x, product=ba.BA_PRODUCT_FULL, **kw)
    return (i["iters"], i["status"], i["relres"])


@pytest.mark.parametrize("give_up", [1, 2])
@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("name", ["tiny", "300"])
def test_solve_given_up(monkeypatch, name, form, give_up):
    """The first solve gives up and is repeated, the second knows better: the
    same bits, without a start and with one that the result replaces."""
    s = SCENES[name]()
    for guess in (False, True):
        ctx = _context(monkeypatch, s, give_up)
        try:
            n = _form(ctx, s)
            g = np.random.default_rng(7).standard_normal((n, 9)) * 1e-3
            x, y = T(g, torch.float64), T(g, torch.float64)
            i1 = _solve(ctx, x, x0=x if guess else None, max_iter=3000, **FORMS[form])
            i2 = _solve(ctx, y, x0=y if guess else None, max_iter=3000, **FORMS[form])
        finally:
            ba.ba_destroy(ctx)
        assert i1 == i2 and i1[1] == 0
        assert torch.equal(x, y)


@pytest.mark.parametrize("give_up", [1, 2])
@pytest.mark.parametrize("opts", [dict(pcg_tol=1e-10), dict(), dict(pcg_tol=1e-10, deflate=True),
                                  dict(pcg_tol=1e-10, precond=ba.BA_PRECOND_FSAI), dict(pcg_tol=1e-10, retriangulate=2)])
def test_step_given_up(monkeypatch, opts, give_up):
    """A step whose solve gives up takes the step of the repeated solve, once:
    the parameters, the state and the report are those of a context that
    solves with one kernel per phase from the start; so is the next step."""
    s = SCENES["300"]()
    got = []
    for warned in (False, True):
        ctx = _context(monkeypatch, s, give_up)
        try:
            if warned:   # a solve that gives up beforehand
                n = _form(ctx, s)
                _solve(ctx, torch.zeros((n, 9), dtype=torch.float64, device="cuda"), tol=1e-10)
            cams, pts, st = T(s.cams_init, torch.float64), T(s.pts_init, torch.float64), ba.new_lm_state(1e-3)
            reports = []
            for _ in range(2):
                info = ba.ba_lm_step(ctx, cams, pts, st, **opts)
                reports.append({k: v for k, v in info.items() if not k.startswith("ms_")})
            got.append((reports, cams, pts, (st.lam, st.nu, st.iter, st.flags)))
        finally:
            ba.ba_destroy(ctx)
    a, b = got
    assert a[0] == b[0] and a[3] == b[3] and a[0][0]["accepted"] == 1
    assert torch.equal(a[1], b[1]) and torch.equal(a[2], b[2])


@pytest.mark.parametrize("name", [n for n in ordered.SCENES if "not taken" not in n])
@pytest.mark.parametrize("fp32", [False, True])
def test_ordered_solve_bit_for_bit(monkeypatch, name, fp32):
    """Above a tolerance of 1e-8, one kernel and one kernel per phase: the same
    iterates, count and residual."""
    s = ordered.SCENES[name]()
    got = []
    for give_up in (None, 1):
        ctx = _context(monkeypatch, s, give_up)
        try:
            n = _form(ctx, s)
            if give_up == 1:
                _solve(ctx, torch.zeros((n, 9), dtype=torch.float64, device="cuda"), tol=1e-6)
            res = []
            for kw in (dict(tol=1e-6, max_iter=3000), dict(tol=1e-7, max_iter=8), dict(tol=1e-7, max_iter=1)):
                x = torch.full((n, 9), 7.0, dtype=torch.float64, device="cuda")
                res.append((_solve(ctx, x, solver_fp32=fp32, **kw), x))
            x = res[1][1].clone()
            res.append((_solve(ctx, x, x0=x, solver_fp32=fp32, tol=1e-3, max_iter=3000), x))
            got.append(res)
        finally:
            ba.ba_destroy(ctx)
    for (ia, xa), (ib, xb) in zip(*got):
        assert ia == ib
        assert torch.equal(xa, xb)


@pytest.mark.parametrize("form", [f for f in FORMS if f != "loose"])
@pytest.mark.parametrize("name", SCENES)
def test_iterates_of_the_tight_solve(monkeypatch, name, form):
    """At 1e-8 and below the sums have another order: after eight iterations
    (damping 1e-2, a condition of a few thousand) the iterates agree to 1e-10,
    from no start and from one."""
    s = SCENES[name]()
    got = []
    for give_up in (None, 1):
        ctx = _context(monkeypatch, s, give_up)
        try:
            n = _form(ctx, s)
            g = T(np.random.default_rng(7).standard_normal((n, 9)) * 1e-3, torch.float64)
            kw = dict(FORMS[form], max_iter=8)
            res = []
            for x0 in (None, g):
                x = torch.zeros((n, 9), dtype=torch.float64, device="cuda")
                res.append((_solve(ctx, x, x0=x0, **kw), x))
            got.append(res)
        finally:
            ba.ba_destroy(ctx)
    for (ia, xa), (ib, xb) in zip(*got):
        assert ia[:2] == ib[:2]
        assert float((xa - xb).norm()) <= 1e-10 * float(xb.norm())
