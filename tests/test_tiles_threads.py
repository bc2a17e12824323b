"""Tile lists do not depend on the number of host threads that build them (patch lists are built by two,
beside the rest of a setup, tile lists by up to eight)."""
import os
import shutil
import subprocess

import pytest

from mginputs import configs as C, hierarchy as H
from tests.test_tiles_host import _ell

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2608_29082_amd", "csrc")


@pytest.mark.parametrize("mesh,KM,side", [("square", 3, 12), ("square", 8, 8), ("lshape", 2, 12), ("lshape", 3, 6)])
def test_lists_are_the_same_for_any_thread_count(tmp_path, mesh, KM, side):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    h = H.square_hierarchy(129) if mesh == "square" else H.lshape_hierarchy(C.rng(7, 4, 0), 120, 4)
    exe = str(tmp_path / "tiles_threads")
    subprocess.run([cxx, "-O1", "-std=c++17", "-pthread", "-I", CSRC,
                    os.path.join(HERE, "native", "tiles_threads.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe, _ell(h.A[0], str(tmp_path)), str(KM), str(side)], capture_output=True, text=True,
                         timeout=120)
    assert out.returncode == 0 and out.stdout.startswith("ok"), (out.returncode, out.stdout, out.stderr)
