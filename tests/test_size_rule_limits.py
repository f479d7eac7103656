"""The size rules' limits, found through the host-only query: the kernel
variant changes exactly where it was measured to (MiB per direction; real
input: MiB of reals, forward and inverse plans apart), and each choice exists
for both signs."""
import pytest

from paper_2203_09384_amd import api

# length -> [(limit in MiB, (ept, wg, variant) up to it)], then the default
C32 = {
    256: [(14, (8, 64, 6)), (16, (16, 128, 12)), (32, (8, 64, 6)), (None, (16, 128, 12))],
    512: [(15, (8, 64, 6)), (None, (8, 64, 12))],
    1024: [(24, (8, 128, 2)), (128, (8, 256, 3)), (None, (16, 64, 3))],
    2048: [(24, (8, 256, 2)), (None, (8, 256, 3))],
    4096: [(16, (8, 512, 2)), (None, (8, 512, 3))],
    8192: [(32, (16, 512, 2)), (None, (16, 512, 3))],
}
R32 = {
    (32, -1): [(32, (4, 128, 7)), (None, (4, 256, 2))],
    (64, +1): [(32, (4, 256, 7)), (None, (8, 256, 3))],
    (256, -1): [(24, (8, 256, 6)), (96, (4, 256, 7)), (None, (8, 256, 6))],
    (256, +1): [(24, (8, 256, 6)), (36, (4, 256, 7)), (None, (8, 256, 6))],
    (512, -1): [(18, (8, 128, 6)), (None, (16, 256, 3))],
    (512, +1): [(24, (8, 128, 6)), (None, (16, 256, 3))],
    (1024, -1): [(32, (8, 64, 6)), (192, (8, 256, 7)), (None, (16, 256, 3))],
    (2048, +1): [(24, (8, 128, 2)), (96, (8, 256, 3)), (None, (16, 64, 3))],
    (4096, -1): [(28, (8, 256, 2)), (None, (16, 128, 3))],
    (4096, +1): [(32, (8, 256, 2)), (None, (16, 128, 3))],
    (8192, -1): [(32, (8, 512, 2)), (None, (8, 512, 3))],
}


def chosen(n, batch, sign, dtype):
    d = api.query(n, batch, sign, dtype)
    return d["ept"], d["wg"], d["variant"]


def check(n, sign, dtype, rows, elem):
    low = 0
    for mib, want in rows:
        first = (low << 20) // (n * elem) + 1 if low else 1
        last = (mib if mib else 2 * low) * (1 << 20) // (n * elem)
        for batch in (first, (first + last) // 2, last):
            assert chosen(n, batch, sign, dtype) == want, (n, batch, sign)
        low = mib


@pytest.mark.parametrize("n", C32)
@pytest.mark.parametrize("sign", [-1, 1])
def test_complex(n, sign):
    check(n, sign, "c32", C32[n], 8)


@pytest.mark.parametrize("n,sign", R32)
def test_real(n, sign):
    check(n, sign, "r32", R32[n, sign], 4)
