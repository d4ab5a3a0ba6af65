"""GPU: the mesh-gradient control's two refilling forms (a branch after each step, branch-free pairs) give the same
scores: the path count decides the form, a path's numbers do not depend on it."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("score", [W.SCORE_EXTEND, W.SCORE_BRIDGE])
@pytest.mark.parametrize("K,t,last,stride,few,many", [
    (65, 0.2, 0.7, 2, 70, 48000),
    (200, 0.1, 1.0, 2, 70, 48000),         # pairs at few paths, branches at many
    (301, 0.02, 0.4, 20, 70, 48000),
    (1000, 0.01, 1.0, 1 << 20, 70, 10000),  # branches where all paths are held at once by that form only
    (1001, 0.02, 0.7, 100, 70, 9000),
])
def test_forms_agree(fk, score, K, t, last, stride, few, many):
    import torch
    G = 48
    x = np.arange(G + 1) / G
    X, Y = np.meshgrid(x, x)
    gx = (X + 0.02 * np.sin(np.pi * X) * np.sin(2 * np.pi * Y)).ravel()
    gy = (Y + 0.015 * np.sin(2 * np.pi * X) * np.sin(np.pi * Y)).ravel()
    grids = (torch.tensor(gx, device="cuda"), torch.tensor(gy, device="cuda"))
    bdry = W.DATA_GRID if score == W.SCORE_BRIDGE else W.DATA_IDENTITY
    data = W.Data(init_kind=W.DATA_GRID, bdry_kind=bdry, score_mode=score, grid_xi=gx, grid_eta=gy)
    pts = np.concatenate([W.uniform_points(27, seed=2, lo=0.02, hi=0.98), [(0.0, 0.3), (1.0, 1.0), (0.5, 1e-9)]])
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    many = many * cus // 256
    dt = t / (K - 1 + last)
    for dens in (W.moving_bump(), W.two_bumps(W.TIME_FROZEN, 0.2)):
        kw = dict(stride=stride, seed=4, plain=False, form=fk.FK_CV_MARTINGALE_GRID, grids=grids, cv_scores=True,
                  exit_step=True)
        small = fk.fk_interface_solve_cv(dens, data, pts, t, dt, few, None, **kw)
        big = fk.fk_interface_solve_cv(dens, data, pts, t, dt, many, None, **kw)
        torch.cuda.synchronize()
        assert torch.equal(big["cv_scores"][:, :few], small["cv_scores"])
        assert torch.equal(big["exit_step"][:, :few], small["exit_step"])
        es = big["exit_step"]
        assert int(big["total_steps"][0]) == int(torch.where(es < 0, K, es).sum())
        # fixed-point sums: 2^-49 per score
        mean = big["cv_scores"].double().mean(1)
        assert (big["xi"] - mean[:, 0]).abs().max() < 1e-12 and (big["eta"] - mean[:, 1]).abs().max() < 1e-12
