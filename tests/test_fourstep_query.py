"""What the query reports for the four-step lengths is what their launches
use: tiles of 8 while there are fewer than 8192 inner transforms, 16 above and
in streams, 32 points per thread from 512 points up (from 128 in large calls),
and the passes with the split for real input above 2^15."""
import numpy as np
import pytest

from paper_2203_09384_amd import api


def passes(n, batch, sign=-1, dtype="c32"):
    d = api.query(n, batch, sign, dtype)
    assert int(np.prod(d["radices"])) == (n if dtype == "c32" else n // 2)
    return (d["ept"], d["wg"], d["transforms_per_wg"], d["grid"]), d["radices"]


@pytest.mark.parametrize("n,batch,want,radices", [
    (1 << 20, 1, (32, 256, 8, 128), [32, 32, 32, 32]),
    (1 << 20, 7, (32, 256, 8, 896), [32, 32, 32, 32]),     # 7168 columns
    (1 << 20, 8, (32, 512, 16, 512), [32, 32, 32, 32]),    # 8192
    (1 << 20, 33, (32, 512, 16, 33 * 64), [32, 32, 32, 32]),
    (1 << 18, 1, (32, 128, 8, 64), [16, 32, 16, 32]),
    (1 << 18, 16, (32, 256, 16, 512), [16, 32, 16, 32]),
    (1 << 17, 8, (32, 128, 8, 256), [16, 32, 16, 16]),     # 8 MiB: 16 points per thread in the row pass
    (1 << 17, 64, (32, 256, 16, 1024), [16, 32, 8, 32]),
    (1 << 16, 4, (16, 256, 16, 64), [16, 16, 16, 16]),
    (1 << 16, 65, (32, 128, 16, 65 * 16), [8, 32, 8, 32]),
    (1 << 15, 4, (16, 256, 16, 32), [16, 16, 2, 8, 8]),
    (1 << 15, 256, (32, 128, 16, 2048), [8, 32, 4, 32]),
    (1 << 15, 320, (16, 256, 16, 2560), [16, 16, 2, 8, 8]),  # 80 MiB
])
def test_complex(n, batch, want, radices):
    assert passes(n, batch) == (want, radices)


@pytest.mark.parametrize("n,batch,sign,want,radices", [
    (1 << 17, 1, -1, (16, 256, 16, 16), [16, 16, 8, 32]),
    (1 << 17, 1, +1, (32, 64, 8, 32), [8, 32, 16, 16]),
    (1 << 21, 1, -1, (32, 256, 8, 128), [32, 32, 32, 32]),
    (1 << 21, 1, +1, (32, 256, 8, 128), [32, 32, 32, 32]),
    (1 << 20, 64, -1, (32, 512, 16, 64 * 32), [32, 32, 16, 32]),
    (1 << 20, 64, +1, (32, 512, 16, 64 * 32), [32, 32, 16, 32]),
])
def test_real(n, batch, sign, want, radices):
    assert passes(n, batch, sign, "r32") == (want, radices)


def test_lds_fits():
    for L in range(15, 21):
        for batch in (1, 3, 40, 300, 3000):
            assert 0 < api.query(1 << L, batch, -1, "c32")["lds_bytes"] <= 160 * 1024
            for sign in (-1, 1):
                assert 0 < api.query(2 << L, batch, sign, "r32")["lds_bytes"] <= 160 * 1024
