"""Axis passes of 512, 1024 and 2048 points (tiles of 16 transforms) where
tiles are ragged: counts that fill no tile, one that leaves a remainder, and
strides below, at and above the tile's 16 transforms.  Against the FP64
oracle; bar, as for every FP32 transform: relative L2 <= 1e-5."""
import numpy as np
import pytest

import oracle
from paper_2203_09384_amd import api, synth
from gpu_util import need_gpu, per_transform_relerr, to_cpu, to_gpu

pytestmark = pytest.mark.gpu
TOL = 1e-5


@pytest.mark.parametrize("n", [512, 1024, 2048])
@pytest.mark.parametrize("lead,stride,batch", [((), 2, 1), ((), 2, 9), ((), 16, 1), ((), 32, 3), ((2,), 4, 3),
                                               ((4,), 64, 1)])
@pytest.mark.parametrize("sign", [-1, 1])
def test_wide_axis(n, lead, stride, batch, sign):
    shape = lead + (n, stride)
    x = synth.uniform_complex(71, (batch,) + shape, key=(n, stride, batch, sign + 1))
    print(f"[case] wide axis shape={shape} batch={batch} sign={sign}", flush=True)
    y = to_cpu(api.PlanND(shape, batch, sign).execute(to_gpu(x)))
    ref = oracle.fftn(x.astype(np.complex128), len(shape), sign, 1.0 if sign < 0 else 1.0 / np.prod(shape))
    assert per_transform_relerr(y.reshape(batch, -1), ref.reshape(batch, -1)) <= TOL


@pytest.mark.parametrize("n,stride,batch", [(128, 2, 16387), (128, 64, 513), (256, 2, 8195), (256, 8, 2051)])
@pytest.mark.parametrize("sign", [-1, 1])
def test_bulk_axis(n, stride, batch, sign):
    """Axes of 128 and 256 points just above the size at which they take 32
    points per thread, with a last tile that is not full."""
    x = synth.uniform_complex(73, (batch, n, stride), key=(n, stride, sign + 1))
    print(f"[case] bulk axis n={n} stride={stride} batch={batch} sign={sign}", flush=True)
    y = to_cpu(api.PlanND((n, stride), batch, sign).execute(to_gpu(x)))
    at = [0, 1, batch // 2, batch - 2, batch - 1]
    ref = oracle.fftn(x[at].astype(np.complex128), 2, sign, 1.0 if sign < 0 else 1.0 / (n * stride))
    assert per_transform_relerr(y[at].reshape(5, -1), ref.reshape(5, -1)) <= TOL
