"""GPU: a node with a score that is not finite or beyond the estimator's bound gets NaN results, on every path kernel
(nodes without one keep theirs)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

BOUND = 512.0            # scores from here on are not summed
G = 32


def _grids(value):
    import torch
    x = np.arange(G + 1) / G
    X, Y = np.meshgrid(x, x)
    gx = X + 0.02 * np.sin(np.pi * X) * np.sin(2 * np.pi * Y)
    gy = Y + 0.015 * np.sin(2 * np.pi * X) * np.sin(np.pi * Y)
    gx[16, 8] = value                     # at (0.25, 0.5)
    return gx, gy, (torch.tensor(gx.ravel(), device="cuda"), torch.tensor(gy.ravel(), device="cuda"))


def _nodes():
    # in the cells around the value, within a few steps of them, and far away
    near = [(0.25, 0.5), (0.24, 0.51), (0.27, 0.5), (0.25, 0.54)]
    return np.array(near + [(0.7, 0.2), (0.8, 0.8), (0.6, 0.5), (0.02, 0.03)])


def _check(g, scores, far=4):
    s = scores.cpu().numpy().astype(np.float64)
    bad = ~(np.abs(s) < BOUND).all(axis=(1, 2))
    assert bad.any() and not bad[far:].any()
    for k in ("xi", "eta", "se_xi", "se_eta"):
        assert np.array_equal(np.isnan(g[k].cpu().numpy()), bad), k
    mean = s[~bad].mean(1)
    assert np.abs(g["xi"].cpu().numpy()[~bad] - mean[:, 0]).max() < 1e-12
    assert np.abs(g["eta"].cpu().numpy()[~bad] - mean[:, 1]).max() < 1e-12


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf, 1e30])
@pytest.mark.parametrize("K,score", [(20, W.SCORE_EXTEND), (48, W.SCORE_EXTEND), (100, W.SCORE_EXTEND),
                                     (20, W.SCORE_BRIDGE), (100, W.SCORE_BRIDGE), (20, W.SCORE_EXPONENTIAL)])
def test_grid_data(fk, K, score, value):
    import torch
    gx, gy, grids = _grids(value)
    bdry = W.DATA_IDENTITY if score == W.SCORE_EXTEND else W.DATA_GRID
    data = W.Data(init_kind=W.DATA_GRID, bdry_kind=bdry, score_mode=score, grid_xi=gx.ravel(), grid_eta=gy.ravel())
    g = fk.fk_interface_solve(W.two_bumps(W.TIME_FROZEN, 0.2), data, _nodes(), 1e-4, 1e-4 / K, 500, seed=3,
                              scores=True, grids=grids)
    torch.cuda.synchronize()
    _check(g, g["scores"])


@pytest.mark.parametrize("value", [np.nan, np.inf, 1e30])
@pytest.mark.parametrize("K,n", [(20, 500), (48, 500), (100, 500), (1200, 100), (20, 40000)])
def test_mesh_gradient_control(fk, K, n, value):
    import torch
    gx, gy, grids = _grids(value)
    data = W.Data(init_kind=W.DATA_GRID, score_mode=W.SCORE_EXTEND, grid_xi=gx.ravel(), grid_eta=gy.ravel())
    g = fk.fk_interface_solve_cv(W.two_bumps(W.TIME_FROZEN, 0.2), data, _nodes(), 1e-4, 1e-4 / K, n, None, stride=2,
                                 seed=3, plain=False, form=fk.FK_CV_MARTINGALE_GRID, grids=grids, cv_scores=True)
    torch.cuda.synchronize()
    _check(g, g["cv_scores"])


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("K", [20, 48, 100])
def test_grid_density(fk, K, value):
    """A density sample that is not finite spoils the drift around it: paths there carry NaN to their scores, and do
    not count as having left the square."""
    import torch
    x = torch.arange(G + 1, dtype=torch.float64, device="cuda") / G
    wg = (1.0 + torch.exp(-((x[None, :] - 0.6) ** 2 + (x[:, None] - 0.4) ** 2) / 0.02)).contiguous()
    wg[16, 8] = value
    g = fk.fk_interface_solve(fk.GridDensity(wg), W.Data(init_kind=W.DATA_SIN), _nodes(), 1e-4, 1e-4 / K, 500, seed=3,
                              scores=True, exit_step=True)
    torch.cuda.synchronize()
    _check(g, g["scores"])
    spoilt = ~np.isfinite(g["scores"].cpu().numpy()).all(-1)
    assert spoilt.any() and (g["exit_step"].cpu().numpy()[spoilt] == -1).all()
