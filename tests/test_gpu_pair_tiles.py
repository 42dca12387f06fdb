"""The pair stage above and below the size from which its work is ordered and
cut by tiles of points (4 GiB of records), with two and with three LDS
buffers (units of fewer and of more than 16 steps), free and fixed cameras
(needs a GPU): RCS and right-hand side against the oracle."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2307_08383_amd import scenegen

from gpu_util import T, block_errors, create

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ba = pytest.importorskip("paper_2307_08383_amd.ba")


@pytest.mark.parametrize("nx,ny,n_pts,n_fixed,precision", [
    (20, 15, 750_000, 0, 0),       # 576 MB of FP64 records: whole pairs, long units
    (50, 40, 750_000, 7, 0),       # short units
    (20, 15, 1_500_000, 7, 1),     # 576 MB of FP32 records
    (60, 50, 5_700_000, 7, 0),     # 4.4 GB: tiles
])
def test_rcs_against_the_oracle(nx, ny, n_pts, n_fixed, precision):
    """About four records a point.  Bounds of the formation tests: blocks
    1e-10 (FP64) and 1e-4 (FP32 records), right-hand side 1e-9 and 1e-4."""
    s = scenegen.aerial_grid_scene(seed=13, nx=nx, ny=ny, n_pts=n_pts, with_stats=False)
    s.cam_fixed[3:3 + n_fixed] = 1
    uv = orc.observations(s)
    P = orc.Problem.from_scene(s, uv)
    P.linearize(s.cams_init, s.pts_init)
    P.form_rcs(1e-2)
    blk_ref, rhs_ref = P.rcs()
    rp, ci = P.pattern()
    ctx = create(s, uv, precision)
    try:
        ba.ba_linearize(ctx, T(s.cams_init, torch.float64), T(s.pts_init, torch.float64))
        ba.ba_form_rcs(ctx, 1e-2)
        blk, rhs = ba.ba_get_rcs(ctx)
        first = blk.copy()
        ba.ba_form_rcs(ctx, 1e-2)
        assert np.array_equal(first, ba.ba_get_rcs(ctx)[0])
    finally:
        ba.ba_destroy(ctx)
    errs, _ = block_errors(blk, blk_ref, rp, ci)
    assert errs.max() <= (1e-10 if precision == 0 else 1e-4)
    rerr = np.linalg.norm(rhs - rhs_ref, axis=1) / np.maximum(np.linalg.norm(rhs_ref, axis=1), 1e-300)
    assert rerr.max() <= (1e-9 if precision == 0 else 1e-4)
