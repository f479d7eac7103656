"""CPU check of the map that deals the tiles of a real-input call to the XCDs:
every tile of every transform exactly once, and all tiles of a transform on one
XCD while 8 transforms are left to deal."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2203_09384_amd", "csrc")


@pytest.fixture(scope="module")
def tm(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("tm") / "libtiles.so")
    r = subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-fPIC", "-shared", f"-I{CSRC}",
                        os.path.join(HERE, "host", "tile_maps_check.cpp"), "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return ctypes.CDLL(out)


@pytest.mark.parametrize("batch", [1, 2, 7, 8, 9, 15, 16, 17, 64, 67])
@pytest.mark.parametrize("per", [4, 8, 16, 64, 128])
def test_deal(tm, batch, per):
    b = np.full(batch * per, -1, np.int64)
    tile = np.full(batch * per, -1, np.int64)
    p = ctypes.POINTER(ctypes.c_int64)
    tm.tm_deal(ctypes.c_int64(batch), ctypes.c_int64(per), b.ctypes.data_as(p), tile.ctypes.data_as(p))
    assert b.min() >= 0 and b.max() < batch and tile.min() >= 0 and tile.max() < per
    assert len(np.unique(b * per + tile)) == batch * per
    whole = batch // 8 * 8
    xcd = np.arange(batch * per) % 8
    for t in range(whole):
        assert len(np.unique(xcd[b == t])) == 1
