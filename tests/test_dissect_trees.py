"""The nested-dissection trees that the library accepts can be launched: every box's front fits what its level's
kernel holds, and every such kernel is compiled (CPU; the library's own tree, its boxes derived anew)."""
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.join(os.path.dirname(HERE), "paper_1402_0266_amd")


@pytest.fixture(scope="module")
def trees(tmp_path_factory):
    hipcc = shutil.which("hipcc")
    if hipcc is None:
        pytest.skip("hipcc not available")
    lib = os.path.join(PKG, "libfk.so")
    if not os.path.exists(lib):
        import __graft_entry__
        __graft_entry__.build()
    exe = str(tmp_path_factory.mktemp("nd") / "nd_trees")
    subprocess.run([hipcc, "-x", "hip", "--cuda-host-only", "-std=c++17", "-O1", "-I", os.path.join(PKG, "csrc"),
                    os.path.join(HERE, "helpers", "nd_trees.cpp"), "-x", "none", lib, "-Wl,-rpath," + PKG, "-o", exe],
                   check=True, capture_output=True)

    def run(shapes):
        text = "\n".join(" ".join(str(int(v)) for v in s) for s in shapes)
        out = subprocess.run([exe], input=text + "\n", capture_output=True, text=True, check=True).stdout
        return np.array([[int(v) for v in ln.split()] for ln in out.strip().splitlines()], dtype=np.int64)
    return run


def _shapes(blocks):
    """Both orientations of every size with a shorter side of at most 127 unknowns (the longer one odd sizes only
    past 300)."""
    longs = [b for b in range(1, 2000) if b <= 300 or b % 37 == 0]
    s = [(a, b) for a in range(1, 128) for b in longs if b >= a]
    # largest pivot count and largest rim of a level from different boxes: 54 + 140 and the like
    s += [(70, 212), (65, 252), (76, 164), (77, 156)]
    return [(a, b, blocks) for a, b in s] + [(b, a, blocks) for a, b in s]


@pytest.mark.parametrize("blocks", [1, 3, 64])
def test_every_accepted_tree_can_be_launched(trees, blocks):
    r = trees(_shapes(blocks))
    bad = r[r[:, 4] == 0]
    assert len(bad) == 0, bad[:8]
    assert (r[:, 3] == 1).sum() > 10000 and r[r[:, 3] == 1, 6].max() == 192
