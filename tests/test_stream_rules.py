"""CPU checks of the rules on the sizes of calls (csrc/stream.hpp): the chunks
of a multidimensional transform cover its batch, none but the last exceeds a
chunk, and no short one is left over."""
import ctypes
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2203_09384_amd", "csrc")
I64 = ctypes.c_int64


@pytest.fixture(scope="module")
def st(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("st") / "libstream.so")
    r = subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-fPIC", "-shared", f"-I{CSRC}",
                        os.path.join(HERE, "host", "stream_check.cpp"), "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    lib = ctypes.CDLL(out)
    for f in ("st_chunk_bytes", "st_tail_bytes", "st_chunk_units", "st_next_chunk"):
        getattr(lib, f).restype = I64
    lib.st_chunk_units.argtypes = [I64]
    lib.st_next_chunk.argtypes = [I64, I64, I64]
    return lib


def chunks(st, count, each, share):
    """Sizes of the chunks of `count` units of `each` bytes; share: the bytes
    of a chunk that a unit takes, in units of its own."""
    per = st.st_chunk_units(share * each)
    got, b = [], 0
    while b < count:
        here = st.st_next_chunk(count - b, per, each)
        assert here >= 1
        got.append(here)
        b += here
    assert b == count
    return per, got


@pytest.mark.parametrize("share", [1, 2])
@pytest.mark.parametrize("log2_each", [15, 16, 20, 22, 23, 24, 25, 26, 28, 29])
def test_chunks(st, share, log2_each):
    each = 1 << log2_each
    tail, whole = st.st_tail_bytes(), st.st_chunk_bytes() // share
    per = st.st_chunk_units(share * each)
    counts = {1, 2, 3, per, per + 1, 2 * per - 1, 2 * per, 2 * per + 1, 5 * per + 3}
    counts |= {per + max(1, tail // each) + d for d in (-1, 0, 1)}
    for count in sorted(c for c in counts if c >= 1):
        per, got = chunks(st, count, each, share)
        assert all(c == per for c in got[:-1])
        assert got[-1] * each <= max(whole, each) + tail
        if len(got) > 1 and got[-1] < per:
            assert got[-1] * each > tail


@pytest.mark.parametrize("log2n", [15, 16, 17])
def test_fourstep_bulk(st, log2n):
    """32 points per thread: never in small calls, always in streams, and at
    2^15 not between 64 MiB and a stream."""
    for f in (st.st_bulk_bytes, st.st_stream_bytes):
        f.restype = I64
    st.st_fourstep_bulk.argtypes = [ctypes.c_int, I64]
    bulk, stream = st.st_bulk_bytes(), st.st_stream_bytes()
    for nbytes, want in ((0, False), (bulk, False), (bulk + 1, True), (stream // 2, True),
                         (stream // 2 + 1, log2n != 15), (stream, log2n != 15), (stream + 1, True)):
        assert bool(st.st_fourstep_bulk(log2n, nbytes)) == want, nbytes


@pytest.mark.parametrize("log2n,most", [(1, 224), (8, 224), (9, 256), (11, 256)])
def test_keep_gradient(st, log2n, most):
    st.st_keep_gradient.argtypes = [ctypes.c_int, I64, ctypes.c_int]
    for nbytes, alone, scaled in ((1 << 10, True, True), (2 << 20, True, True), ((2 << 20) + 8, False, False),
                                  (32 << 20, False, False), ((32 << 20) + 8, False, True), (most << 20, False, True),
                                  ((most << 20) + 8, False, False), (1 << 30, False, False)):
        assert bool(st.st_keep_gradient(log2n, nbytes, 0)) == alone, nbytes
        assert bool(st.st_keep_gradient(log2n, nbytes, 1)) == scaled, nbytes


@pytest.mark.parametrize("log2n,low,high", [(1, 8, 20), (7, 6, 20), (8, 8, 20), (12, 8, 28), (14, 8, 20)])
def test_feed_next(st, log2n, low, high):
    st.st_feed_next.argtypes = [ctypes.c_int, I64]
    for mib, extra, want in ((0, 8, True), (low, 0, True), (low, 8, False), (16, 0, False), (high, 0, False),
                             (high, 8, True), (256, 0, True)):
        assert bool(st.st_feed_next(log2n, (mib << 20) + extra)) == want, (mib, extra)
