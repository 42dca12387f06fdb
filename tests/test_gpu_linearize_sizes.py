"""Linearization and point stage where their waves and workgroups are partly
filled (needs a GPU): observation counts around 64 and 256 and their
multiples; Jacobians, residuals, RCS and point terms against the oracle."""
import dataclasses

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2307_08383_amd import scenegen

from gpu_util import T, check_against_oracle, create

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ba = pytest.importorskip("paper_2307_08383_amd.ba")


def _scene(n_obs):
    """12 cameras, whole tracks taken until n_obs observations."""
    s = scenegen.aerial_grid_scene(seed=14, nx=4, ny=3, n_pts=2000, with_stats=False)
    length = np.bincount(s.obs_pt, minlength=s.n_pts)
    take, left = np.zeros(s.n_pts, bool), n_obs
    for p in range(s.n_pts):
        if length[p] == left or length[p] <= left - 2:
            take[p] = True
            left -= length[p]
    assert left == 0
    keep = take[s.obs_pt]
    new_id = np.cumsum(take) - 1
    return dataclasses.replace(s, n_pts=int(take.sum()), n_obs=n_obs, pts_true=s.pts_true[take], pts_init=s.pts_init[take],
                               obs_cam=s.obs_cam[keep], obs_pt=new_id[s.obs_pt[keep]].astype(np.int32),
                               noise=np.ascontiguousarray(s.noise[:, keep]))


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n_obs", [96, 97, 127, 128, 129, 255, 256, 257, 289, 1023, 4097])
def test_against_the_oracle(n_obs, precision):
    """Damping 1, so that systems of few observations are well conditioned;
    bounds of the fused path's test."""
    s = _scene(n_obs)
    uv = orc.observations(s)
    P = orc.Problem.from_scene(s, uv)
    ctx = create(s, uv, precision)
    try:
        cost = ba.ba_linearize(ctx, T(s.cams_init, torch.float64), T(s.pts_init, torch.float64))
        ba.ba_form_rcs(ctx, 1.0)
        F_ref, *_ = check_against_oracle(ctx, P, s.cams_init, s.pts_init, 1.0, precision, np.random.default_rng(1))
    finally:
        ba.ba_destroy(ctx)
    assert abs(cost - F_ref) <= 1e-10 * F_ref
