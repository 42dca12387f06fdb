"""The end of an LM step, decided on the device (needs a GPU): the reported
decision is the one its figures call for, a step that is not accepted leaves
the parameters bit for bit, an accepted one moves them to the reported cost,
a linearization out of range changes nothing, and the stages' times add up."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2307_08383_amd import scenegen

from gpu_util import T, create

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ba = pytest.importorskip("paper_2307_08383_amd.ba")

OPTS = [dict(), dict(precond=ba.BA_PRECOND_FSAI), dict(deflate=True), dict(product=ba.BA_PRODUCT_UPPER), dict(retriangulate=2),
        dict(pcg_max_iter=0), dict(pcg_max_iter=1)]


@pytest.mark.parametrize("opts", OPTS)
@pytest.mark.parametrize("spread", [0.0, 0.4])
def test_decision_and_update(opts, spread):
    """40 steps: to convergence, where cost no longer falls, and from points
    that lie far off, whose first steps overshoot."""
    s = scenegen.aerial_grid_scene(seed=15, nx=5, ny=4, n_pts=400, with_stats=False)
    uv = orc.observations(s)
    rng = np.random.default_rng(2)
    ctx = create(s, uv)
    try:
        cams, pts = T(s.cams_init, torch.float64), T(s.pts_init + spread * rng.standard_normal(s.pts_init.shape), torch.float64)
        st = ba.new_lm_state(1e-4)
        last = None
        for _ in range(40):
            c0, p0 = cams.clone(), pts.clone()
            info = ba.ba_lm_step(ctx, cams, pts, st, **opts)
            want = (info["pcg_status"] in (ba.BA_OK, 4) and info["model_decrease"] > 0 and np.isfinite(info["cost_new"]) and
                    info["cost_new"] < info["cost"])
            assert info["accepted"] == int(want)
            if last is not None:
                assert abs(info["cost"] - last) <= 1e-11 * last
            if want:
                last = info["cost_new"]
            else:
                assert torch.equal(cams, c0) and torch.equal(pts, p0)
                last = info["cost"]
            parts = sum(info[k] for k in ("ms_linearize", "ms_form_rcs", "ms_pcg", "ms_back_substitute", "ms_evaluate"))
            assert info["ms_form_rcs"] > 0 and info["ms_pcg"] > 0 and info["ms_back_substitute"] > 0 and info["ms_evaluate"] > 0
            assert parts <= info["ms_total"] * 1.001 and info["ms_total"] < 1000
    finally:
        ba.ba_destroy(ctx)


def test_out_of_range_changes_nothing():
    s = scenegen.aerial_grid_scene(seed=15, nx=5, ny=4, n_pts=400, with_stats=False)
    uv = orc.observations(s)
    ctx = create(s, uv)
    try:
        bad = s.pts_init.copy()
        bad[7, 0] = np.nan
        cams, pts = T(s.cams_init, torch.float64), T(bad, torch.float64)
        st = ba.new_lm_state(1e-4)
        with pytest.raises(ba.BAError):
            ba.ba_lm_step(ctx, cams, pts, st)
        assert np.array_equal(cams.cpu().numpy(), s.cams_init)
        assert np.array_equal(pts.cpu().numpy(), bad, equal_nan=True)
        assert st.iter == 0 and st.lam == 1e-4
        good = T(s.pts_init, torch.float64)
        assert ba.ba_lm_step(ctx, cams, good, st)["accepted"] == 1
    finally:
        ba.ba_destroy(ctx)
