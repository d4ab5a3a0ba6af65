"""GPU: the refilling kernel's few-steps form (33 to 64 steps over a horizon that paths leave in) and the short-horizon
kernel against the branch-free pairs of a batch, bitwise."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _nodes():
    p = W.uniform_points(21, seed=11, lo=0.001, hi=0.999)
    return np.concatenate([p, [(0.0, 0.5), (1.0, 1.0), (-0.0, 0.25), (0.5, 1e-9), (1.0 - 1e-9, 0.5), (0.02, 0.03)]])


def _density(fk, name):
    if name != "grid":
        return {"const": W.CONST, "bump": W.static_bump(), "moving": W.moving_bump(),
                "two_frozen": W.two_bumps(W.TIME_FROZEN, 0.2), "ring": W.paper_ring(W.TIME_BACKWARD),
                "ridge": W.ridge()}[name]
    return fk.GridDensity(fk.fk_density_sample(W.two_bumps(W.TIME_FROZEN, 0.2), 0.2, 40))


def _compare(fk, dens, t, K, last, n, data, plans, pts=None):
    import torch
    dt, pts = t / (K - 1 + last), _nodes() if pts is None else pts
    b = fk.FkBatch([(dens, t, data.t_init, pts, 5)], data, dt, n, seed=77)
    ref = b.run(exit_step=True, scores=True)
    for plan in plans:
        out = fk.fk_interface_solve(dens, data, pts, t, dt, n, seed=77, level_id=5, exit_step=True, scores=True,
                                    steps=True, plan=plan)
        torch.cuda.synchronize()
        for k in ("xi", "eta", "se_xi", "se_eta", "exit_step", "scores", "total_steps"):
            assert np.array_equal(out[k].cpu().numpy(), ref[k].cpu().numpy()), (k, plan)
        es = ref["exit_step"].cpu().numpy()
        assert np.array_equal(out["steps"].cpu().numpy(), np.where(es < 0, K, es).sum(1))
    b.close()


@pytest.mark.parametrize("name", ["const", "bump", "moving", "two_frozen", "ring", "ridge", "grid"])
@pytest.mark.parametrize("K,t,last,n", [(33, 0.1, 1.0, 65), (33, 0.1, 0.4, 2), (48, 0.3, 1.0, 300), (63, 3.0, 0.7, 129),
                                        (64, 0.06, 1.0, 257), (64, 0.2, 0.5, 1000)])
def test_few_steps_form(fk, name, K, t, last, n):
    dens = _density(fk, name)
    for data in (W.Data(t_init=0.1), W.Data(init_kind=W.DATA_SIN, bdry_kind=W.DATA_SIN),
                 W.Data(bdry_kind=W.DATA_ZERO, score_mode=W.SCORE_PROJECT)):
        _compare(fk, dens, t, K, last, n, data, (None, {"chunk": 1}, {"chunk": 100, "block": 64},
                                                 {"blocks_per_cu": 1, "node_tile": 4}))


@pytest.mark.parametrize("K,t,last", [(1, 5e-4, 1.0), (20, 1e-3, 1.0), (19, 0.2, 0.3), (32, 0.1, 0.7)])
def test_short_horizons_with_a_grid_density(fk, K, t, last):
    _compare(fk, _density(fk, "grid"), t, K, last, 130, W.Data(init_kind=W.DATA_SIN), (None, {"chunk": 1}))


def _near_sides(t):
    p = W.uniform_points(24, seed=3)
    d = np.sqrt(0.31 * t)
    p[:8, 0] = np.linspace(0.0, 1.2 * d, 8)           # around the line from which lanes take other paths
    p[8:16, 1] = 1.0 - np.linspace(0.0, 1.2 * d, 8)
    p[16:20] = [(0.0, 0.0), (1.0, 0.5), (0.5, 1e-9), (d, 0.5)]
    return p


@pytest.mark.parametrize("name", ["const", "moving", "two_frozen", "ring", "grid"])
@pytest.mark.parametrize("K,t,last,n", [(33, 0.05, 1.0, 2), (33, 0.01, 0.4, 63), (48, 0.02, 1.0, 64), (63, 0.05, 0.7, 65),
                                        (64, 1e-3, 1.0, 300), (64, 0.05, 0.5, 2100)])
def test_nodes_near_a_side(fk, name, K, t, last, n):
    p = _near_sides(t)
    for data in (W.Data(t_init=0.1), W.Data(init_kind=W.DATA_SIN, bdry_kind=W.DATA_ZERO)):
        _compare(fk, _density(fk, name), t, K, last, n, data, (None, {"chunk": 1}, {"chunk": 100, "block": 64},
                                                              {"chunk": 2048}), p)


@pytest.mark.parametrize("name", ["const", "moving", "two_frozen", "ring", "grid"])
@pytest.mark.parametrize("K,t,last,n", [(33, 0.05, 1.0, 16385), (64, 0.05, 0.5, 16385), (64, 1e-3, 1.0, 16450),
                                        (48, 0.02, 1.0, 16384), (32, 0.05, 1.0, 16450)])
def test_nodes_near_a_side_with_many_paths(fk, name, K, t, last, n):
    """Past 32 steps, with more rounds of 64 paths than wavefronts fit (24 nodes x 256 on this GPU), the
    short-horizon kernel lets the lanes of nodes near a side take other paths of a chunk."""
    _compare(fk, _density(fk, name), t, K, last, n, W.Data(init_kind=W.DATA_SIN, bdry_kind=W.DATA_ZERO),
             (None, {"chunk": 64}, {"chunk": 65}, {"chunk": 1000, "block": 64}, {"chunk": 2048}), _near_sides(t))
