"""GPU: a path's control-variate score does not depend on which lanes of its
wavefront hold paths (the network evaluation takes those lanes only), on its
place in the launch, or on how the horizon cuts its pairs of steps."""
import numpy as np
import pytest

import oracle.mlp as M
import workloads as W

pytestmark = pytest.mark.gpu


def _params(seed):
    rng = np.random.default_rng(seed)
    return (W.mlp_init(seed) * 2.5 + 0.05 * rng.standard_normal(M.N_PARAMS)).astype(np.float32)


@pytest.mark.parametrize("form,precision,score", [("dynkin", "split", None), ("martingale", "split", None),
                                                  ("martingale", "bf16", None),
                                                  ("martingale", "bf16", W.SCORE_BRIDGE)])
@pytest.mark.parametrize("K,last,stride", [(1, 1.0, 2), (40, 1.0, 4), (41, 0.4, 10)])
def test_scores_do_not_depend_on_the_launch(fk, form, precision, score, K, last, stride):
    import torch
    t = 0.02
    dt = t / (K - 1 + last)
    dens = W.moving_bump()
    pts = np.concatenate([W.uniform_points(5, seed=2, lo=0.05, hi=0.95), [(0.01, 0.5), (0.5, 0.995), (0.0, 0.2)]])
    data = W.Data() if score is None else W.Data(score_mode=score)
    cv = fk.FkCv(_params(1), 0.1, grad_precision=precision)
    kw = dict(stride=stride, seed=4, form=fk.FK_CV_DYNKIN if form == "dynkin" else fk.FK_CV_MARTINGALE, exit_step=True,
              cv_scores=True)

    def run(n, plan=None):
        g = fk.fk_interface_solve_cv(dens, data, pts, t, dt, n, cv, plan=plan, **kw)
        torch.cuda.synchronize()
        return {k: v.cpu().numpy() for k, v in g.items() if not k.startswith("_")}

    full = run(130)
    assert np.isfinite(full["cv_scores"]).all()
    assert int(full["total_steps"][0]) == np.where(full["exit_step"] < 0, K, full["exit_step"]).sum()
    assert ((full["exit_step"] >= -1) & (full["exit_step"] <= K)).all()
    for n in (2, 15, 16, 17, 33, 49, 64, 65):
        for plan in (None, {"chunk": 1}, {"chunk": 7, "block": 64}):
            g = run(n, plan)
            assert np.array_equal(g["cv_scores"], full["cv_scores"][:, :n]), (n, plan)
            assert np.array_equal(g["exit_step"], full["exit_step"][:, :n]), (n, plan)
    cv.close()


@pytest.mark.parametrize("score", [W.SCORE_EXTEND, W.SCORE_BRIDGE])
@pytest.mark.parametrize("K,last,stride", [(65, 1.0, 2), (100, 0.3, 10), (101, 1.0, 1 << 20)])
def test_mesh_control_scores_do_not_depend_on_the_launch(fk, score, K, last, stride):
    """The same for the mesh's gradient over longer horizons, whose lanes start their paths at once."""
    import torch
    G = 20
    x = np.arange(G + 1) / G
    X, Y = np.meshgrid(x, x)
    gx = (X + 0.02 * np.sin(np.pi * X) * np.sin(2 * np.pi * Y)).ravel()
    gy = (Y + 0.015 * np.sin(2 * np.pi * X) * np.sin(np.pi * Y)).ravel()
    grids = (torch.tensor(gx, device="cuda"), torch.tensor(gy, device="cuda"))
    bdry = W.DATA_GRID if score == W.SCORE_BRIDGE else W.DATA_IDENTITY
    data = W.Data(init_kind=W.DATA_GRID, bdry_kind=bdry, score_mode=score, grid_xi=gx, grid_eta=gy)
    pts = np.concatenate([W.uniform_points(5, seed=2, lo=0.05, hi=0.95), [(0.01, 0.5), (1.0, 1.0), (0.0, 0.2)]])
    t = 0.1
    dt = t / (K - 1 + last)

    def run(n, plan=None):
        g = fk.fk_interface_solve_cv(W.moving_bump(), data, pts, t, dt, n, None, stride=stride, seed=4, plain=False,
                                     form=fk.FK_CV_MARTINGALE_GRID, grids=grids, cv_scores=True, exit_step=True,
                                     plan=plan)
        torch.cuda.synchronize()
        return {k: v.cpu().numpy() for k, v in g.items() if not k.startswith("_")}

    full = run(130)
    assert np.isfinite(full["cv_scores"]).all()
    assert int(full["total_steps"][0]) == np.where(full["exit_step"] < 0, K, full["exit_step"]).sum()
    for n in (2, 17, 64, 65):
        for plan in (None, {"chunk": 1}, {"chunk": 7, "block": 64}):
            g = run(n, plan)
            assert np.array_equal(g["cv_scores"], full["cv_scores"][:, :n]), (n, plan)
            assert np.array_equal(g["exit_step"], full["exit_step"][:, :n]), (n, plan)
