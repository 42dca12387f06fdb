"""The FSAI factor's kernel over the sizes of its local matrices (needs a GPU):
fully connected blocks of 4 to 36 cameras, so sets of 1, 2, ... up to the
largest of 28 members, against the oracle."""
import numpy as np
import pytest

from paper_2307_08383_amd import scenegen

from test_gpu_fsai import CAP, _case, _oracle_fsai

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
ba = pytest.importorskip("paper_2307_08383_amd.ba")


@pytest.mark.parametrize("n_grid", [2, 3, 4, 5, 6])
def test_factor(n_grid):
    """FP32 local factorisation: block error (Frobenius) up to 1e-4 of the
    block, as in the factor's parity test."""
    s = scenegen.tiny_scene(seed=8, n_grid=n_grid, n_pts=1500, t_hi=min(10, n_grid * n_grid), with_stats=False)
    P, ctx = _case(s)
    try:
        dxc = torch.empty((P.n_rows, 9), dtype=torch.float64, device="cuda")
        assert ba.ba_pcg_solve(ctx, dxc, tol=1e-10, max_iter=3000, precond=ba.BA_PRECOND_FSAI)["status"] == 0
        G = ba.ba_get_fsai(ctx).astype(np.float64)
    finally:
        ba.ba_destroy(ctx)
    _, _, _, _, _, Gs, J = _oracle_fsai(P, s)
    assert sorted({len(j) for j in J}) == list(range(1, min(P.n_rows, CAP + 1) + 1))
    for k in range(len(Gs)):
        scale = np.linalg.norm(Gs[k])
        assert np.linalg.norm(G[k] - Gs[k]) <= 1e-4 * scale
