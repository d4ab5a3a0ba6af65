"""GPU: the short-horizon path kernel against the refilling one, bitwise.

A batch of one level runs the refilling kernel at any step count; a single
solve of at most 32 steps (64 on a short horizon) runs the lockstep kernel.
Both draw the same numbers and sum exactly, so every output is the same."""
import math

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

DENSITIES = {
    "const": W.CONST,
    "bump": W.static_bump(),
    "ridge": W.ridge(),
    "moving": W.moving_bump(),
    "moving_frozen": W.moving_bump(W.TIME_FROZEN, 0.3),
    "two": W.two_bumps(W.TIME_BACKWARD),
    "two_frozen": W.two_bumps(W.TIME_FROZEN, 0.2),
    "ring": W.paper_ring(W.TIME_BACKWARD),
    "ring_frozen": W.paper_ring(W.TIME_FROZEN, 0.1),
}


def _nodes():
    # interior, on and next to the boundary, a negative zero
    p = W.uniform_points(21, seed=11, lo=0.001, hi=0.999)
    return np.concatenate([p, [(0.0, 0.5), (1.0, 1.0), (-0.0, 0.25), (0.5, 1e-9), (1.0 - 1e-9, 0.5)]])


def _same(single, batch, keys):
    import torch
    torch.cuda.synchronize()
    for k in keys:
        a, b = single[k].cpu().numpy(), batch[k].cpu().numpy()
        assert np.array_equal(a, b), f"{k}: {np.abs(a.astype(np.float64) - b).max()}"


@pytest.mark.parametrize("name", sorted(DENSITIES))
@pytest.mark.parametrize("K,t,last", [(1, 5e-4, 1.0), (2, 1e-3, 1.0), (19, 1e-3, 0.3), (20, 0.4, 1.0), (32, 0.1, 0.7),
                                      (63, 0.03, 1.0), (64, 0.05, 0.5)])
def test_equals_the_refilling_kernel(name, K, t, last):
    import paper_1402_0266_amd as fk
    dens, pts = DENSITIES[name], _nodes()
    dt = t / (K - 1 + last)
    n = {1: 2, 2: 63, 19: 64, 20: 65, 32: 257, 63: 127, 64: 300}[K]
    for data in (W.Data(t_init=0.1), W.Data(init_kind=W.DATA_SIN, bdry_kind=W.DATA_SIN),
                 W.Data(bdry_kind=W.DATA_ZERO, score_mode=W.SCORE_PROJECT)):
        b = fk.FkBatch([(dens, t, data.t_init, pts, 5)], data, dt, n, seed=77)
        ref = b.run(exit_step=True, scores=True)
        for plan in (None, {"chunk": 1}, {"chunk": 100, "block": 64}, {"blocks_per_cu": 1, "node_tile": 4}):
            out = fk.fk_interface_solve(dens, data, pts, t, dt, n, seed=77, level_id=5, exit_step=True, scores=True,
                                        steps=True, plan=plan)
            _same(out, ref, ("xi", "eta", "se_xi", "se_eta", "exit_step", "scores", "total_steps"))
            steps = np.where(ref["exit_step"].cpu().numpy() < 0, K, ref["exit_step"].cpu().numpy()).sum(1)
            assert np.array_equal(out["steps"].cpu().numpy(), steps)
        b.close()


@pytest.mark.parametrize("K,last,t", [(0, 1.0, 0.0), (1, 1.0, 0.3), (3, 0.4, 0.2), (33, 1.0, 0.04), (33, 0.6, 0.04)])
def test_pairs_cut_by_the_horizon(K, last, t):
    """Odd step counts, no steps at all, and steps long enough to jump far past the square, in the refilling kernel
    (which takes steps in pairs) against the lockstep one."""
    import paper_1402_0266_amd as fk
    pts = np.concatenate([_nodes(), [(1.0, 0.3), (0.3, 1.0), (0.7, -0.0)]])
    dt = t / (K - 1 + last) if K else 0.01
    for name in ("const", "moving", "two"):
        for data in (W.Data(t_init=0.1), W.Data(init_kind=W.DATA_SIN, bdry_kind=W.DATA_ZERO)):
            b = fk.FkBatch([(DENSITIES[name], t, data.t_init, pts, 5)], data, dt, 129, seed=7)
            ref = b.run(exit_step=True, scores=True)
            out = fk.fk_interface_solve(DENSITIES[name], data, pts, t, dt, 129, seed=7, level_id=5, exit_step=True,
                                        scores=True)
            _same(out, ref, ("xi", "eta", "se_xi", "se_eta", "exit_step", "scores", "total_steps"))
            b.close()


def test_mask_and_nodes_outside():
    """Masked nodes get the full solve's results, others keep their values; a node outside the square gets NaN."""
    import torch

    import paper_1402_0266_amd as fk
    dens, pts = W.two_bumps(W.TIME_FROZEN, 0.2), _nodes()
    pts = np.concatenate([pts, [(1.5, 0.5), (math.nan, 0.5)]])
    data, n = W.Data(), 130
    full = fk.fk_interface_solve(dens, data, pts, 1e-3, 5e-5, n, seed=3, steps=True)
    xi = full["xi"].cpu().numpy()
    assert np.isnan(xi[-2:]).all() and np.isfinite(xi[:-2]).all()
    assert int(full["total_steps"]) == int(full["steps"].sum()) and (full["steps"][-2:] == 0).all()
    for keep in (np.zeros(len(pts)), np.ones(len(pts)), np.arange(len(pts)) % 3 == 0):
        mask = keep.astype(np.uint8)
        out = {k: torch.full((len(pts),), -7.0, dtype=torch.float64, device="cuda") for k in ("xi", "eta", "se_xi", "se_eta")}
        out["total_steps"] = torch.zeros(1, dtype=torch.int64, device="cuda")
        fk.fk_interface_solve(dens, data, pts, 1e-3, 5e-5, n, seed=3, out=out, mask=mask)
        for k in ("xi", "eta", "se_xi", "se_eta"):
            want = np.where(mask != 0, full[k].cpu().numpy(), -7.0)
            assert np.array_equal(out[k].cpu().numpy(), want, equal_nan=True)
        assert int(out["total_steps"]) == int(full["steps"].cpu().numpy()[mask != 0].sum())


@pytest.mark.parametrize("K,stride,n", [(1, 2, 2), (2, 2, 65), (31, 4, 70), (32, 20, 130)])
def test_mesh_gradient_form(oracle_mod, K, stride, n):
    """Ragged step and path counts of the mesh-gradient control against the oracle, with and without the gradient
    table.  As in test_gpu_cv.py a path may sit on the other side of a cell edge in FP32: such scores are bounded by
    1e-3, the others agree to 1e-6."""
    import torch

    import paper_1402_0266_amd as fk
    G = 24
    x = np.arange(G + 1) / G
    X, Y = np.meshgrid(x, x)
    gx = X + 0.02 * np.sin(np.pi * X) * np.sin(2 * np.pi * Y)
    gy = Y + 0.015 * np.sin(2 * np.pi * X) * np.sin(np.pi * Y)
    data = W.Data(init_kind=W.DATA_GRID, score_mode=W.SCORE_EXTEND, grid_xi=gx.ravel(), grid_eta=gy.ravel())
    dens, pts = W.two_bumps(W.TIME_FROZEN, 0.2), W.uniform_points(9, seed=4, lo=0.01, hi=0.99)
    t = 2e-3
    grids = (torch.tensor(gx.ravel(), device="cuda"), torch.tensor(gy.ravel(), device="cuda"))
    o = oracle_mod.fk_solve_cv(dens, data, pts, t, t / K, n, seed=9, uhat=oracle_mod.UHAT_GRID, stride=stride,
                               form=oracle_mod.CV_MARTINGALE, want_scores=True, want_exit=True)
    got = []
    for table in (True, False):
        ws = None if table else torch.empty(fk.library().fk_interface_cv_workspace_bytes(len(pts), n),
                                            dtype=torch.uint8, device="cuda")
        g = fk.fk_interface_solve_cv(dens, data, pts, t, t / K, n, None, stride=stride, seed=9, plain=False,
                                     form=fk.FK_CV_MARTINGALE_GRID, grids=grids, cv_scores=True, exit_step=True,
                                     workspace=ws, grad_table=table)
        torch.cuda.synchronize()
        got.append({k: v.cpu().numpy() for k, v in g.items() if not k.startswith("_")})
    for k in got[0]:
        assert np.array_equal(got[0][k], got[1][k]), k
    assert np.array_equal(got[0]["exit_step"], o["exit_step"])
    ds = np.abs(got[0]["cv_scores"].astype(np.float64) - o["cv_scores"]).max(-1)
    assert np.mean(ds < 1e-6) >= 0.99 and ds.max() < 1e-3
    assert int(got[0]["total_steps"][0]) == np.where(o["exit_step"] < 0, K, o["exit_step"]).sum()


@pytest.mark.parametrize("G,t,K,last,stride", [(24, 2e-3, 20, 1.0, 2), (99, 1e-3, 9, 0.4, 2), (100, 1e-3, 12, 1.0, 4),
                                               (200, 0.012, 20, 1.0, 2), (768, 5e-4, 19, 0.7, 2)])
def test_mesh_gradient_from_a_tile(G, t, K, last, stride):
    """Many paths at many nodes read the mesh's gradient from LDS (the whole mesh, one that just fits, ones cut by the
    tile, with paths that leave it), few paths from memory: the same paths have bitwise the same scores, and the
    larger solve's sums are those of its scores."""
    import torch

    import paper_1402_0266_amd as fk
    x = np.arange(G + 1) / G
    X, Y = np.meshgrid(x, x)
    gx = X + 0.02 * np.sin(np.pi * X) * np.sin(2 * np.pi * Y)
    gy = Y + 0.015 * np.sin(2 * np.pi * X) * np.sin(np.pi * Y)
    data = W.Data(init_kind=W.DATA_GRID, score_mode=W.SCORE_EXTEND, grid_xi=gx.ravel(), grid_eta=gy.ravel())
    grids = (torch.tensor(gx.ravel(), device="cuda"), torch.tensor(gy.ravel(), device="cuda"))
    pts = np.concatenate([W.uniform_points(592, seed=8, lo=0.0, hi=1.0),
                          [(0.0, 0.0), (1.0, 1.0), (0.5, 1e-9), (1.0 - 1e-9, 0.5), (1.5, 0.5)]])
    dt, n, few = t / (K - 1 + last), 17000, 96
    mask = (np.arange(len(pts)) % 64 != 3).astype(np.uint8)
    for dens in (W.two_bumps(W.TIME_FROZEN, 0.2), W.moving_bump()):
        for m in (None, mask):
            kw = dict(stride=stride, seed=9, plain=False, form=fk.FK_CV_MARTINGALE_GRID, grids=grids, cv_scores=True,
                      exit_step=True, mask=m)
            big = fk.fk_interface_solve_cv(dens, data, pts, t, dt, n, None, **kw)
            small = fk.fk_interface_solve_cv(dens, data, pts, t, dt, few, None, **kw)
            torch.cuda.synchronize()
            on = np.ones(len(pts), bool) if m is None else m != 0
            on[-1] = False
            sel = torch.tensor(on, device="cuda")
            assert torch.equal(big["cv_scores"][sel, :few], small["cv_scores"][sel])
            assert torch.equal(big["exit_step"][sel, :few], small["exit_step"][sel])
            es = big["exit_step"][sel]
            assert int(big["total_steps"][0]) == int(torch.where(es < 0, K, es).sum())
            # fixed-point sums: 2^-49 per score
            mean = big["cv_scores"][sel].double().mean(1)
            assert (big["xi"][sel] - mean[:, 0]).abs().max() < 1e-12
            assert (big["eta"][sel] - mean[:, 1]).abs().max() < 1e-12
