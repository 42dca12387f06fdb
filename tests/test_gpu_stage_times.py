"""The stage times of the last formation stay what they were when the
parameters are linearized again (needs a GPU), after an LM step, whose
linearization and point stage are one kernel, and after ba_form_rcs."""
import pytest

from oracle import oracle as orc
from paper_2307_08383_amd import scenegen

from gpu_util import T, create

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ba = pytest.importorskip("paper_2307_08383_amd.ba")


@pytest.mark.parametrize("fused", [True, False])
def test_a_later_linearization_leaves_them(fused):
    s = scenegen.aerial_grid_scene(seed=15, nx=10, ny=8, n_pts=8000, with_stats=False)
    ctx = create(s, orc.observations(s))
    try:
        cams, pts = T(s.cams_init, torch.float64), T(s.pts_init, torch.float64)
        if fused:
            ba.ba_lm_step(ctx, cams, pts, ba.new_lm_state(1e-4))
        else:
            ba.ba_linearize(ctx, cams, pts)
            ba.ba_form_rcs(ctx, 1e-4)
        before = ba.ba_get_stage_ms(ctx)
        assert before[0] > 0 and before[2] > 0 and before[3] > 0
        assert (before[1] == 0) == fused   # the fused point stage is part of the linearization
        ba.ba_linearize(ctx, cams, pts)
        after = ba.ba_get_stage_ms(ctx)
        assert after[1:] == before[1:] and after[0] > 0
    finally:
        ba.ba_destroy(ctx)
