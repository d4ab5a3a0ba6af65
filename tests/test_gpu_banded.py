"""GPU: the banded elimination of the sub-domain solves where it is still taken -- sub-domains whose dissection would
have too large a front, and workspaces of the banded size that are too small for the dissection -- against the oracle;
the equidistributed edge data of long edges."""
import ctypes
import math

import numpy as np
import pytest

import oracle.subdomain as S
import workloads as W

pytestmark = pytest.mark.gpu

DENS = W.Density(W.KIND_BUMP, amp=2.0, width2=0.04, cx=0.4, cy=0.6)   # drift in both directions


def _align(n):
    return (n + 255) // 256 * 256


def _banded_bytes(px, py, N):
    """Workspace of the banded elimination: U rows, y, coefficients and right-hand sides both ways, separators, edges."""
    q, long = min(N // px, N // py) - 1, max(N // px, N // py) - 1
    blocks, n = px * py, q * long
    row = q + 1 if q + 1 in (8, 12, 16, 20, 24, 32) else 16 * ((q + 31) // 16)
    sep = 2 * (q * q + 2 * q) + 2 * q
    parts = (blocks * n * row, 2 * blocks * n, 8 * blocks * n, 4 * blocks * n, blocks * sep, 4 * N)
    return sum(_align(8 * p) for p in parts)


def _solve(fk, px, py, N, size, steady=False):
    import torch
    x = np.arange(N + 1) / N
    X, Y = np.meshgrid(x, x)
    xi0 = X + 0.02 * np.sin(math.pi * X) * np.sin(2 * math.pi * Y)
    eta0 = Y + 0.015 * np.sin(2 * math.pi * X) * np.sin(math.pi * Y)
    ij = S.interface_index_rect(px, py, N)
    rng = np.random.default_rng(1000 * px + N)
    ix = xi0[ij[:, 1], ij[:, 0]] + 1e-3 * rng.standard_normal(len(ij))
    iy = eta0[ij[:, 1], ij[:, 0]] + 1e-3 * rng.standard_normal(len(ij))
    dev = [torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda") for a in (xi0, eta0, ix, iy)]
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    out = torch.empty((2, N + 1, N + 1), dtype=torch.float64, device="cuda")
    d = fk._density(DENS)
    rc = fk.library().subdomain_solve_rect(ctypes.byref(d), 0.0, 1e-3, px, py, N, 0, dev[0].data_ptr(),
                                           dev[1].data_ptr(), dev[2].data_ptr(), dev[3].data_ptr(), out[0].data_ptr(),
                                           out[1].data_ptr(), ws.data_ptr(), size, fk._stream(torch, out.device))
    torch.cuda.synchronize()
    if rc != fk.FK_OK:
        return rc, math.nan
    ox, oy = S.subdomain_be_step_rect(DENS, 0.0, 1e-3, px, py, N, xi0, eta0, ix, iy)
    g = out.cpu().numpy()
    return rc, max(np.abs(g[0] - ox).max(), np.abs(g[1] - oy).max())


# Both eliminations meet at a separator (two workgroups a sub-domain).
@pytest.mark.parametrize("px,py,N", [
    (1, 2, 140),                          # 139 x 69 unknowns: a window of 96
    (1, 2, 192), (2, 1, 230),             # 191 x 95; 114 x 229: windows of 112 and 144
    (1, 2, 226), (1, 2, 256), (2, 1, 256),   # 225 x 112, 255 x 127, 127 x 255: 128 and 144
    (1, 4, 280),                          # 279 x 69, four sub-domains
])
def test_fronts_too_large(fk, px, py, N):
    need = fk.subdomain_workspace_bytes_rect(px, py, N)
    assert need == _banded_bytes(px, py, N)           # nothing is asked for a dissection
    rc, err = _solve(fk, px, py, N, need)
    assert rc == fk.FK_OK and err < 1e-12
    assert _solve(fk, px, py, N, need - 256)[0] == fk.FK_E_NOMEM


@pytest.mark.parametrize("px,py,N", [
    (17, 8, 136), (3, 2, 36),             # 8 x 17 and 12 x 18 cells: from one end, one wavefront
    (8, 1, 64), (2, 1, 24), (1, 2, 24),   # 8 x 64, 12 x 24, 24 x 12: from both ends
    (2, 1, 32), (2, 1, 40), (2, 1, 48), (8, 1, 256),   # windows of 16, 20, 24, 32
])
def test_workspace_of_the_banded_size(fk, px, py, N):
    size = _banded_bytes(px, py, N)
    assert fk.subdomain_workspace_bytes_rect(px, py, N) > size      # the dissection takes more
    rc, err = _solve(fk, px, py, N, size)
    assert rc == fk.FK_OK and err < 1e-12
    assert _solve(fk, px, py, N, size - 256)[0] == fk.FK_E_NOMEM


@pytest.mark.parametrize("N", [255, 256, 257, 300, 513, 768])
def test_equidistributed_edges_in_runs(fk, N):
    """Edges of more than 256 cells are summed in runs of several cells: the boundary nodes against quadrature of w."""
    import torch
    dens = W.moving_bump(W.TIME_FROZEN, 0.1)
    out = torch.full((2, N + 1, N + 1), -7.0, dtype=torch.float64, device="cuda")
    ws = torch.empty(max(fk.fk_boundary_workspace_bytes(N), 256), dtype=torch.uint8, device="cuda")
    fk.fk_boundary_data(dens, 0.1, N, W.DATA_EQUIDISTRIBUTED, out[0], out[1], workspace=ws)
    torch.cuda.synchronize()
    g = out.cpu().numpy()
    inner = g[:, 1:-1, 1:-1]
    assert (inner == -7.0).all()
    for k in {0, 1, 2, 3, N // 3, N // 2, 255, 256, N - 2, N - 1, N} & set(range(N + 1)):
        s = k / N
        for edge, row in ((0.0, 0), (1.0, N)):
            assert abs(g[0, row, k] - S._edge_equidistribution(dens, 0.1, s, edge, True)) < 1e-9
            assert abs(g[1, k, row] - S._edge_equidistribution(dens, 0.1, s, edge, False)) < 1e-9
    assert (g[0, :, 0] == 0).all() and (g[0, :, -1] == 1).all() and (g[1, 0] == 0).all() and (g[1, -1] == 1).all()
