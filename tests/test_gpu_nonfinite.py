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


DEGENERATE = {
    # w = 0 at the centre in FP32, and beyond FP32's range: the drift is 0 / 0, 0 inf or inf there
    "zero": W.Density(W.KIND_BUMP, amp=-1 + 1e-10, width2=0.01, cx=0.5, cy=0.5),
    "narrow": W.Density(W.KIND_BUMP, amp=1.0, width2=1e-42, cx=0.5, cy=0.5),
    "steep": W.Density(W.KIND_BUMP, amp=1e38, width2=1e-3, cx=0.5, cy=0.5),
    "moving": W.Density(W.KIND_MOVING_BUMP, amp=1e38, width2=1e-3, cx=0.5, cy=0.5, orbit_r=0.25, omega=6.25),
    "two": W.Density(W.KIND_TWO_BUMPS, amp=-0.5, width2=0.01, cx=0.5, cy=0.5),
    "ridge": W.Density(W.KIND_RIDGE, amp=1e38, width2=1e-3, cx=0.5),
}


@pytest.mark.parametrize("name", sorted(DEGENERATE))
@pytest.mark.parametrize("K,t", [(20, 1e-3), (48, 1e-2), (100, 1e-2), (1200, 1e-2)])
def test_degenerate_analytic_density(fk, name, K, t):
    """A position that is not a number is not an exit (its path runs to the horizon and scores the initial data
    there): the nodes it reaches get NaN, also with boundary data 0."""
    import torch
    data = W.Data(bdry_kind=W.DATA_ZERO)
    pts = np.array([(0.5, 0.5), (0.5, 0.7), (0.01, 0.5), (0.75, 0.5)])
    g = fk.fk_interface_solve(DEGENERATE[name], data, pts, t, t / K, 200, seed=3, scores=True, exit_step=True)
    b = fk.FkBatch([(DEGENERATE[name], t, 0.0, pts, 0)], data, t / K, 200, seed=3)
    r = b.run(scores=True, exit_step=True)
    torch.cuda.synchronize()
    s, e = g["scores"].cpu().numpy(), g["exit_step"].cpu().numpy()
    # the centre: NaN in both coordinates at the first step
    if name in ("zero", "two", "narrow"):
        assert np.isnan(s[0]).all() and (e[0] == -1).all()
    bad = ~np.isfinite(s).all(axis=(1, 2))
    assert np.array_equal(np.isnan(g["xi"].cpu().numpy()), bad) and bad.any()
    assert (s[e >= 0] == 0.0).all()
    for k in ("xi", "eta", "se_xi", "se_eta", "scores", "exit_step", "total_steps"):
        assert np.array_equal(g[k].cpu().numpy(), r[k].cpu().numpy(), equal_nan=True), k
    b.close()
