"""GPU: a plan tuned for one kernel is not handed to another."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def test_tuned_plans_of_two_kernels(fk, tmp_path, monkeypatch):
    """48 steps run the short-horizon kernel over t = 0.01 and the refilling one over t = 0.1."""
    import torch
    cache = tmp_path / "plans"
    monkeypatch.setenv("FK_TUNE_CACHE", str(cache))
    pts = torch.tensor(W.uniform_points(23, seed=6), device="cuda")

    def keys(t, steps=48):
        p = fk.FkPlan()
        p.autotune(W.moving_bump(), W.Data(), pts, t, t / steps, 70)
        torch.cuda.synchronize()
        return [ln.split()[0] for ln in cache.read_text().splitlines()]

    assert len(keys(0.01)) == 1
    both = keys(0.1)
    assert len(both) == 2 and both[0] != both[1]
    # the same kernel and shape: found in the cache
    assert keys(0.02) == both and keys(0.2) == both
