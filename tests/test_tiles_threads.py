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


def _run(tmp_path, name, A, KM, side):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path / name)
    subprocess.run([cxx, "-O1", "-std=c++17", "-pthread", "-I", CSRC, os.path.join(HERE, "native", name + ".cpp"),
                    "-o", exe, "-ldl"], check=True)
    out = subprocess.run([exe, _ell(A, str(tmp_path)), str(KM), str(side)], capture_output=True, text=True,
                         timeout=120)
    assert out.returncode == 0 and out.stdout.startswith("ok"), (out.returncode, out.stdout, out.stderr)


@pytest.mark.parametrize("mesh,KM,side", [("square", 3, 12), ("square", 8, 8), ("lshape", 2, 12), ("lshape", 3, 6)])
def test_lists_are_the_same_for_any_thread_count(tmp_path, mesh, KM, side):
    h = H.square_hierarchy(129) if mesh == "square" else H.lshape_hierarchy(C.rng(7, 4, 0), 120, 4)
    _run(tmp_path, "tiles_threads", h.A[0], KM, side)


def test_threads_or_memory_refused(tmp_path):
    """A worker thread that cannot start, or cannot have its memory, ends neither the process nor the lists'
    order: a setup builds them on its own thread, or runs the level by sweeps."""
    _run(tmp_path, "tiles_refused", H.square_hierarchy(129).A[0], 3, 8)
