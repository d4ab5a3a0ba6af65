"""The sub-domain solve's check |b| h / 2 < 1: refused exactly where a fine
sample of |b| over the distance to the centre refuses it."""
import ctypes
import math

import numpy as np
import pytest

import workloads as W


def _sampled(d):
    """max |b| on the sample that defines the check."""
    if d.kind == W.KIND_RING:
        r = 1.5 * np.arange(1, 20001) / 20000
        e = np.exp(d.width2 * np.abs(r * r - 0.01))
        return (2 * d.amp * abs(d.width2) * r * e / (1 + d.amp * e)).max()
    A, r = abs(d.amp), 4 * math.sqrt(d.width2) * np.arange(1, 4001) / 4000
    e = np.exp(-r * r / d.width2)
    b = (2 * A / d.width2 * r * e / (1 + (A if d.amp >= 0 else -A) * e)).max()
    return 2 * b if d.kind == W.KIND_TWO_BUMPS else b


@pytest.mark.parametrize("kind", [W.KIND_BUMP, W.KIND_RIDGE, W.KIND_MOVING_BUMP, W.KIND_TWO_BUMPS, W.KIND_RING])
def test_refused_as_sampled(kind):
    import paper_1402_0266_amd as fk
    lib, rng, N = fk.library(), np.random.default_rng(kind), 40
    need = lib.subdomain_workspace_bytes(2, 20)
    refused = 0
    for _ in range(60):
        if kind == W.KIND_RING:
            d = W.Density(kind, amp=10 ** rng.uniform(-1, 3), width2=-10 ** rng.uniform(0, 3))
        else:
            amp = 10 ** rng.uniform(-1, 3) if rng.random() < 0.7 else -rng.uniform(0, 0.999)
            d = W.Density(kind, amp=amp, width2=10 ** rng.uniform(-4, 0))
        # scaled towards the edge of the rule
        target = 2.0 * N * (1 + rng.choice([-0.2, -1e-3, -1e-6, 1e-6, 1e-3, 0.2]))
        for _ in range(60):
            s = target / _sampled(d)
            if abs(s - 1) < 1e-12 or not np.isfinite(s):
                break
            d = W.Density(kind, amp=d.amp, width2=d.width2 * (s if kind == W.KIND_RING else s ** -2.0))
        if not 0 < abs(d.width2) < 1e6 or abs(_sampled(d) / (2.0 * N) - 1) < 1e-9:
            continue
        wide = _sampled(d) / (2.0 * N) >= 1
        refused += wide
        # (the arrays are never read: a refused call, or one that finds no device)
        if wide or not _has_device():
            rc = lib.subdomain_solve(ctypes.byref(fk._density(d)), 0.0, 1e-3, 2, 20, 0, 4096, 4096, 4096, 4096, 4096,
                                     4096, 4096, need, None)
            assert rc == (fk.FK_E_UNSUPPORTED if wide else fk.FK_E_NODEVICE), (d, _sampled(d) / (2.0 * N))
    assert refused > 5


def _has_device():
    import torch
    return torch.cuda.is_available()
