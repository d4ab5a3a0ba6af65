"""GPU: the nested-dissection sub-domain solves at the sizes where the tree
changes shape, and the banded elimination where it takes over."""
import ctypes
import math

import numpy as np
import pytest

import oracle.subdomain as S
import workloads as W

pytestmark = pytest.mark.gpu


def _problem(px, py, N, seed=0):
    x = np.arange(N + 1) / N
    X, Y = np.meshgrid(x, x)
    xi0 = X + 0.02 * np.sin(math.pi * X) * np.sin(2 * math.pi * Y)
    eta0 = Y + 0.015 * np.sin(2 * math.pi * X) * np.sin(math.pi * Y)
    ij = S.interface_index_rect(px, py, N)
    rng = np.random.default_rng(seed + 1000 * px + N)
    ix = xi0[ij[:, 1], ij[:, 0]] + 1e-3 * rng.standard_normal(len(ij))
    iy = eta0[ij[:, 1], ij[:, 0]] + 1e-3 * rng.standard_normal(len(ij))
    return xi0, eta0, ix, iy


def _cuda(a):
    import torch
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


# A sub-domain's unknowns are (N/px - 1) x (N/py - 1).
@pytest.mark.parametrize("px,py,N", [
    (1, 1, 2), (1, 1, 3), (2, 3, 6),      # one unknown; two by two; two by one
    (1, 1, 4), (1, 1, 5), (4, 3, 12),     # 9, 16 and 6 unknowns: a leaf, two leaves
    (2, 2, 10), (3, 5, 60),               # 4 x 4; 19 x 11
    (20, 20, 40), (18, 18, 72),           # many sub-domains of one leaf (few are banded)
    (16, 1, 32), (1, 16, 48),             # strips one and two unknowns wide
    (2, 2, 26), (5, 3, 60), (8, 8, 96),   # odd and even halves, few and many sub-domains
    (2, 1, 100), (3, 3, 99), (1, 1, 127), (1, 1, 128),
    (16, 2, 256), (2, 4, 320),
    (1, 4, 256),                          # 255 x 63: banded, the fronts would be too large
])
def test_against_oracle(fk, px, py, N):
    import torch
    # mild drift: |b| h / 2 < 1 on the coarsest grid
    dens = W.ridge(amp=0.5, width2=0.5, cx=0.35) if N < 20 else W.ridge(amp=1.0, width2=0.05)
    xi0, eta0, ix, iy = _problem(px, py, N)
    print(f"[gpu] dissect {px} x {py}, N = {N}", flush=True)
    g = fk.subdomain_solve_rect(dens, 0.0, 1e-3, px, py, N, _cuda(xi0), _cuda(eta0), _cuda(ix), _cuda(iy))
    torch.cuda.synchronize()
    ox, oy = S.subdomain_be_step_rect(dens, 0.0, 1e-3, px, py, N, xi0, eta0, ix, iy)
    assert max(np.abs(g[0].cpu().numpy() - ox).max(), np.abs(g[1].cpu().numpy() - oy).max()) < 1e-12


@pytest.mark.parametrize("px,py,N", [(17, 8, 136)])
def test_workspace_of_the_banded_elimination(fk, px, py, N):
    """A workspace too small for the dissection still solves (banded), to rounding the same; a smaller one is refused."""
    import torch
    lib, dens = fk.library(), W.ridge(amp=1.0, width2=0.05)
    xi0, eta0, ix, iy = (_cuda(a) for a in _problem(px, py, N))
    want = fk.subdomain_solve_rect(dens, 0.0, 1e-3, px, py, N, xi0, eta0, ix, iy)
    need = fk.subdomain_workspace_bytes_rect(px, py, N)
    d = fk._density(dens)

    def solve(size):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        out = torch.empty((2, N + 1, N + 1), dtype=torch.float64, device="cuda")
        rc = lib.subdomain_solve_rect(ctypes.byref(d), 0.0, 1e-3, px, py, N, 0, xi0.data_ptr(), eta0.data_ptr(),
                                      ix.data_ptr(), iy.data_ptr(), out[0].data_ptr(), out[1].data_ptr(),
                                      ws.data_ptr(), size, fk._stream(torch, out.device))
        torch.cuda.synchronize()
        return rc, out

    rc, full = solve(need)
    assert rc == fk.FK_OK and torch.equal(full[0], want[0]) and torch.equal(full[1], want[1])
    rc, small = solve(need - 256)
    assert rc == fk.FK_OK and (small - full).abs().max() < 1e-12
    assert solve(1 << 12)[0] == fk.FK_E_NOMEM


@pytest.mark.parametrize("px,py,N", [(1, 1, 4), (2, 2, 40), (2, 3, 48), (4, 2, 96)])
def test_steady_against_long_step(fk, px, py, N):
    """The steady solve is the limit of a backward-Euler step of length D: they differ by the step's own 1 / D."""
    import torch
    dens = W.ridge(amp=0.5, width2=0.5, cx=0.35)
    xi0, eta0, ix, iy = (_cuda(a) for a in _problem(px, py, N))
    s = fk.subdomain_solve_rect(dens, 0.0, math.inf, px, py, N, None, None, ix, iy)
    b = fk.subdomain_solve_rect(dens, 0.0, 1e9, px, py, N, xi0, eta0, ix, iy)
    torch.cuda.synchronize()
    # |u - u_D| <= |u^n - u| / (D lambda_min), lambda_min > 2, plus rounding (condition number ~ N^2)
    assert max((s[0] - b[0]).abs().max(), (s[1] - b[1]).abs().max()) < 1e-9


@pytest.mark.parametrize("px,py,N", [(3, 1, 213), (1, 3, 213), (2, 1, 154)])
def test_largest_pivots_and_rim_in_different_boxes(fk, px, py, N):
    """Trees with a level whose most pivots and most lines around a box add up to more than any front of it holds
    (70 x 212: 54 + 140; 76 x 153 does not)."""
    import torch
    dens = W.Density(W.KIND_BUMP, amp=2.0, width2=0.04, cx=0.4, cy=0.6)
    xi0, eta0, ix, iy = _problem(px, py, N)
    g = fk.subdomain_solve_rect(dens, 0.0, 1e-3, px, py, N, _cuda(xi0), _cuda(eta0), _cuda(ix), _cuda(iy))
    torch.cuda.synchronize()
    ox, oy = S.subdomain_be_step_rect(dens, 0.0, 1e-3, px, py, N, xi0, eta0, ix, iy)
    assert max(np.abs(g[0].cpu().numpy() - ox).max(), np.abs(g[1].cpu().numpy() - oy).max()) < 1e-12
