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


# (cells a side, sub-domains in x and y, cells of a sub-domain) of large grids: leaves, boxes of level 1 or unknowns
# by the 2^32, and strips with more than 2^15 unknowns a side.
LARGE = [(27456, 8, 11), (16384, 8, 8), (16380, 9, 10), (24576, 12, 12), (65535, 3, 5), (32768, 4, 32768),
         (32768, 32768, 4), (40000, 4, 40000), (32767, 31, 32767)]


@pytest.mark.parametrize("N,mx,my", LARGE)
def test_large_grids(trees, N, mx, my):
    """Accepted only with every launch below 2^32 work-items and unknowns that pack (others take the banded LU)."""
    blocks = (N // mx) * (N // my)
    r = trees([(mx - 1, my - 1, blocks), (my - 1, mx - 1, blocks)])
    assert (r[:, 4] == 1).all(), r


def test_large_grids_that_fit_are_accepted(trees):
    # 8191^2 sub-domains' leaves of 64 work-items; 2^15 - 1 unknowns in a strip
    r = trees([(3, 3, 8191 * 4096), (3, 32767, 128), (7, 7, 2 ** 21)])
    assert (r[:, 3] == 1).all() and (r[:, 4] == 1).all(), r
