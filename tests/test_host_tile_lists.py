"""Gather lists of the tiled edge pass, checked on the host: every list entry is
an entity of the mesh and every stencil operand finds its own, also beside
pentagons, where some slots of the canonical stencil order are empty."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

from synthetic.mesh import icosahedral, planar_hex

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lists(tmp_path_factory):
    from paper_2105_13484_amd import build
    cc = shutil.which("g++")
    if not cc or not os.path.isdir("/opt/rocm/include"):
        pytest.skip("no g++ or HIP headers")
    lib = str(tmp_path_factory.mktemp("tile_lists") / "lists.so")
    cmd = [cc, "-O1", "-std=c++17", "-shared", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", build.CSRC,
           "-o", lib, os.path.join(ROOT, "tests", "host_tile_lists.cpp"), os.path.join(build.CSRC, "sse_mesh.cpp")]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    return ctypes.CDLL(lib, mode=os.RTLD_LAZY)


@pytest.mark.parametrize("make", [lambda: planar_hex(10, 10, 1.0e4), lambda: icosahedral(2), lambda: icosahedral(3)])
@pytest.mark.parametrize("T", [8, 16, 32])
@pytest.mark.parametrize("canonical", [0, 1])
def test_lists_name_the_stencils_operands(lists, make, T, canonical):
    from paper_2105_13484_amd import ssprkse
    mesh = make()
    d, keep = ssprkse.mesh_desc(mesh, np.ones(mesh.nCells), np.ones(mesh.nCells, np.uint8))
    lists.check_tile_lists.restype = ctypes.c_long
    assert lists.check_tile_lists(ctypes.byref(d), T, canonical) == 0
    del keep
