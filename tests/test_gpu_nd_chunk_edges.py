"""Multidimensional transforms in chunks: every array next to a chunk's edge,
with a short last chunk that joins the one before and a longer one of its
own.  Against the FP64 oracle; bar, as for every FP32 transform: relative
L2 <= 1e-5."""
import numpy as np
import pytest
import torch

import oracle
from paper_2203_09384_amd import api
from gpu_util import need_gpu, per_transform_relerr, to_cpu

pytestmark = pytest.mark.gpu
TOL = 1e-5


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


def check(shape, batch, sign, at):
    n = int(np.prod(shape))
    g = torch.Generator(device="cuda").manual_seed(79)
    x = torch.view_as_complex(torch.rand((batch,) + shape + (2,), generator=g, device="cuda").mul_(2).sub_(1))
    print(f"[case] shape={shape} batch={batch} sign={sign}", flush=True)
    y = api.PlanND(shape, batch, sign).execute(x)
    for b in sorted({min(max(a, 0), batch - 1) for a in at}):
        ref = oracle.fftn(to_cpu(x[b:b + 1]).astype(np.complex128), len(shape), sign, 1.0 if sign < 0 else 1.0 / n)
        assert per_transform_relerr(to_cpu(y[b]).reshape(1, -1), ref.reshape(1, -1)) <= TOL, b


# arrays of 4 MiB, 64 to a chunk: one chunk, a joined tail of 1 and of 8
# arrays, a tail of 9 of its own, two chunks and a joined tail
@pytest.mark.parametrize("batch", [64, 65, 72, 73, 129])
@pytest.mark.parametrize("sign", [-1, 1])
def test_images(batch, sign):
    check((512, 1024), batch, sign, [0, 63, 64, 65, 127, 128, batch - 1])


# 256 KiB, 512 to a chunk (the single-pass 2D kernel first): tails of 128
# (joined) and 129 arrays
@pytest.mark.parametrize("batch", [513, 640, 641])
def test_volumes(batch):
    check((32, 32, 32), batch, -1, [0, 511, 512, 513, batch - 1])


# volumes of 2 and 4 planes, which run as one chunk, and of 8, which do not
@pytest.mark.parametrize("shape,batch", [((2, 128, 128), 1100), ((4, 32, 32), 8200), ((8, 64, 64), 1050)], ids=str)
@pytest.mark.parametrize("sign", [-1, 1])
def test_few_planes(shape, batch, sign):
    chunk = (128 << 17) // int(np.prod(shape))
    check(shape, batch, sign, [0, chunk - 1, chunk, 2 * chunk - 1, 2 * chunk, batch - 1])


# four-step last axes: one chunk, chunks with a joined and a separate tail,
# three axes, an array beyond a chunk
@pytest.mark.parametrize("shape,batch", [((32, 65536), 9), ((4, 32768), 258), ((4, 131072), 73), ((2, 8, 32768), 70),
                                         ((2048, 32768), 1)], ids=str)
@pytest.mark.parametrize("sign", [-1, 1])
def test_four_step_last_axis(shape, batch, sign):
    chunk = max(1, (256 << 17) // int(np.prod(shape)))
    check(shape, batch, sign, [0, chunk - 1, chunk, batch - 1])


# sizes at which the first pass's stores change, and one array above
@pytest.mark.parametrize("shape,low,high", [((1024, 32), 8, 20), ((256, 128), 6, 20), ((128, 256), 8, 20),
                                            ((64, 512), 8, 20), ((32, 1024), 8, 20), ((16, 2048), 8, 20),
                                            ((8, 4096), 8, 28), ((4, 16384), 8, 20)], ids=str)
def test_first_pass_stores(shape, low, high):
    n = int(np.prod(shape))
    for mib in (low, high):
        for batch in ((mib << 17) // n, (mib << 17) // n + 1):
            check(shape, batch, -1, [0, batch // 2, batch - 1])
