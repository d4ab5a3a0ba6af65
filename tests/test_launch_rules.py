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
    """A batch's residency goes by the steps of the level its steps are in, not by its longest level."""
    short = " ".join(["50 1521"] * 15)
    long = " ".join(["200 1521"] * 15)
    steps = rules(f"levels {short} 1000 29", f"levels {short} 1600 77", f"levels {long} 4000 29", f"levels {long} 10000 29")
    assert all(v < 1000 for v in steps), steps
    assert rules(*(f"blocks {v} 4 256" for v in steps)) == [0] * 4
    # one level, levels alike, and a ramp whose later levels take most of the steps
    one, alike, ramp = rules("levels 5000 33", "levels 2000 10 2000 99",
                             "levels " + " ".join(f"{100 * i} 381" for i in range(1, 17)))
    assert (one, alike) == (5000, 2000) and 1000 <= ramp < 1600
    assert rules("blocks 5000 4 256", "blocks 2000 4 256", f"blocks {ramp} 4 256", "blocks 5000 40 256") == [3, 4, 4, 0]
    assert rules("levels 0 5", "levels 0 5 1000 5") == [0, 1000]
