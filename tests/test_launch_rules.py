"""Rules that choose a kernel or its residency (CPU; the library's own functions through a small C++ program)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.join(os.path.dirname(HERE), "paper_1402_0266_amd")


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    hipcc = shutil.which("hipcc")
    if hipcc is None:
        pytest.skip("hipcc not available")
    lib = os.path.join(PKG, "libfk.so")
    if not os.path.exists(lib):
        import __graft_entry__
        __graft_entry__.build()
    exe = str(tmp_path_factory.mktemp("rules") / "launch_rules")
    subprocess.run([hipcc, "-x", "hip", "--cuda-host-only", "-std=c++17", "-O1", "-I", os.path.join(PKG, "csrc"), "-I",
                    os.path.join(os.path.dirname(HERE), "include"), os.path.join(HERE, "helpers", "launch_rules.cpp"),
                    "-x", "none", lib, "-Wl,-rpath," + PKG, "-o", exe], check=True, capture_output=True)

    def run(*lines):
        out = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True).stdout
        return [int(v) for v in out.split()]
    return run


def test_one_long_level_does_not_cut_the_residency_of_short_ones(rules):
    """With many paths, a batch's residency goes by the steps of the level its steps are in, not by its longest level."""
    short = " ".join(["50 1521"] * 15)
    long = " ".join(["200 1521"] * 15)
    steps = rules(f"levels {short} 1000 29", f"levels {short} 1600 77", f"levels {long} 4000 29", f"levels {long} 10000 29")
    assert all(v < 1000 for v in steps), steps
    assert rules(*(f"blocks {v} 4000 9 256" for v in steps)) == [0] * 4
    # few paths leave the wavefronts of any form idle: by the longest level
    assert rules(*(f"blocks {v} {k} 8 256" for v in steps for k in (900, 3000, 4000))) == [0, 4, 3] * 4
    # one level, levels alike, and a ramp whose later levels take most of the steps
    one, alike, ramp = rules("levels 5000 33", "levels 2000 10 2000 99",
                             "levels " + " ".join(f"{100 * i} 381" for i in range(1, 17)))
    assert (one, alike) == (5000, 2000) and 1000 <= ramp < 1600
    assert rules("blocks 5000 5000 4 256", "blocks 2000 2000 4 256", f"blocks {ramp} 1600 9 256",
                 "blocks 5000 5000 40 256") == [3, 4, 4, 0]
    assert rules("levels 0 5", "levels 0 5 1000 5") == [0, 1000]


def test_form_of_the_mesh_gradient_control(rules):
    """Branch-free pairs only where they were not slower than a branch after each step."""
    ask = lambda *a, b=0: [divmod(v, 10) for v in rules(*(f"mgg {K} {t} {u} {b}" for K, t, u in a))]
    # few steps; many paths that end all the time
    assert ask((33, 0.3, 1), (64, 0.1, 5), (100, 0.01, 200), (199, 0.1, 13), (400, 0.1, 82), (999, 0.1, 20.5)) == [(0, 0)] * 6
    # all paths held at once by the other form only, and few leaving
    assert ask((64, 1e-3, 4.5), (400, 0.01, 5.2), (1000, 0.01, 5.9), (4000, 0.03, 4.1), (10000, 1e-3, 6.0)) == \
        [(0, 5), (0, 6), (0, 6), (0, 5), (0, 6)]
    assert ask((65, 0.1, 12), (1000, 0.1, 82), (1000, 0.1, 5.2), (2000, 0.01, 3.9), (3999, 0.01, 7)) == [(1, 0)] * 5
    # long horizons: on as many workgroups as hold the paths
    assert ask((4000, 0.01, 1.5), (4000, 0.01, 2.4), (10000, 0.01, 3.6), (4000, 0.01, 7), (10000, 0.1, 6),
               (10000, 0.1, 40)) == [(1, 2), (1, 3), (1, 4), (1, 3), (1, 2), (1, 3)]
    # the bridge test: pairs throughout
    assert ask((33, 0.1, 9), (65, 0.01, 200), (1000, 0.01, 5.2), (4000, 0.01, 4.5), (4000, 0.1, 4.5), b=1) == \
        [(1, 0), (1, 0), (1, 3), (1, 3), (1, 2)]


def test_short_horizon_kernel_with_the_mesh_gradient(rules):
    """Where its lanes neither wait for paths that have left nor for gathers that miss the caches."""
    ask = lambda *a: rules(*("mesh " + " ".join(str(v) for v in q) for q in a))
    #       table, grid, paths, stride, t, K, nodes
    assert ask((1, 768, 16384, 2, 5e-4, 20, 10689), (1, 40, 130, 2, 1e-3, 32, 77), (0, 768, 16384, 2, 5e-4, 20, 10689),
               (0, 64, 4096, 2, 0.05, 32, 1521), (1, 768, 64, 2, 0.05, 32, 1521), (1, 768, 4096, 2, 1e-3, 32, 10689)) == \
        [1] * 6
    # one gather, at the start
    assert ask((0, 768, 4096, 1 << 30, 0.1, 32, 10689), (0, 768, 4096, 32, 0.1, 32, 10689),
               (0, 768, 256, 64, 0.05, 64, 10689), (0, 768, 320, 64, 0.05, 64, 10689)) == [1, 1, 1, 0]
    # past 32 steps: where all paths are under way at once
    assert ask((1, 768, 64, 2, 0.05, 64, 10689), (1, 768, 65, 2, 0.05, 64, 10689), (0, 256, 500, 2, 0.05, 64, 1521),
               (0, 768, 2, 2, 1e-3, 64, 10689), (0, 768, 64, 4, 0.05, 64, 10689), (0, 40, 4096, 2, 0.05, 33, 1521),
               (1, 768, 130, 4, 0.05, 64, 10689), (0, 768, 130, 4, 0.05, 64, 10689)) == [1, 0, 1, 0, 1, 0, 1, 0]
    # paths spread over hundreds of cells; the grids themselves from memory
    assert ask((1, 768, 4096, 2, 0.05, 32, 1521), (1, 768, 4096, 4, 0.05, 32, 1521), (0, 768, 130, 2, 1e-3, 32, 10689),
               (0, 768, 130, 4, 1e-3, 32, 10689), (0, 768, 130, 2, 1e-3, 20, 10689), (0, 768, 500, 2, 1e-3, 20, 10689),
               (0, 768, 2, 2, 1e-3, 32, 10689), (0, 256, 130, 2, 1e-3, 32, 10689), (0, 256, 4096, 2, 0.05, 32, 1521)) == \
        [0, 1, 0, 1, 1, 0, 1, 1, 0]
    assert rules("lockstep 32 3.0 0", "lockstep 64 0.05 2", "lockstep 64 0.06 0", "lockstep 65 0.001 0",
                 "lockstep 20 0.001 3", "lockstep 20 0.001 4") == [1, 1, 0, 0, 0, 0]


def test_grabs_of_the_network_forms_on_few_steps(rules):
    """256 paths a grab where that keeps every wavefront at work."""
    assert rules("network 77 400 0 1", "network 77 1000 0 1", "network 77 4096 0 1", "network 1521 400 0 1",
                 "network 10689 173 0 1", "network 1521 1000 0 1") == [32, 64, 64, 128, 256, 256]
    assert rules("network 77 400 0 0", "network 77 1000 0 0", "network 77 4096 0 0", "network 1521 64 0 0") == \
        [64, 128, 256, 256]
    assert rules("network 616 400 1 1", "network 85512 173 1 1") == [32, 256]
