"""The order in which a launch takes the tiles of C (csrc/tile_order.hpp, plain integer code), compiled for the host."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_every_tile_once_and_panels_shared(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no g++")
    exe = str(tmp_path / "tile_order_check")
    subprocess.run([cxx, "-O2", "-std=c++17", "-Wall", "-D__host__=", "-D__device__=", "-D__forceinline__=inline",
                    os.path.join(HERE, "tile_order_check.cpp"), "-o", exe], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert res.returncode == 0 and "grids ok" in res.stdout, res.stdout
