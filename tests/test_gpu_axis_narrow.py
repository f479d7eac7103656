"""Axes of 2048 points in narrow tiles: counts that fill no tile, short strides
at any count, longer ones on both sides of 1024 and 2048 transforms.  Against the FP64 oracle; bar, as for every FP32 transform:
relative L2 <= 1e-5."""
import numpy as np
import pytest
import torch

import oracle
from paper_2203_09384_amd import api
from gpu_util import need_gpu, per_transform_relerr, to_cpu

pytestmark = pytest.mark.gpu
TOL = 1e-5


@pytest.mark.parametrize("shape,batch", [((2048, 2), 1), ((2048, 2), 3), ((2048, 2), 700), ((2, 2048, 2), 5),
                                         ((2048, 4), 17), ((2048, 16), 1), ((2048, 16), 65), ((2048, 32), 32),
                                         ((2048, 32), 33), ((2048, 32), 64), ((2048, 32), 65), ((2048, 512), 2),
                                         ((2048, 512), 3), ((2048, 2048), 1), ((2048, 16), 128), ((2048, 16), 129), ((2, 2048, 8), 9),
                                         ((2048, 2), 4100)], ids=str)
@pytest.mark.parametrize("sign", [-1, 1])
def test_axis(shape, batch, sign):
    need_gpu()
    n = int(np.prod(shape))
    g = torch.Generator(device="cuda").manual_seed(83)
    x = torch.view_as_complex(torch.rand((batch,) + shape + (2,), generator=g, device="cuda").mul_(2).sub_(1))
    print(f"[case] shape={shape} batch={batch} sign={sign}", flush=True)
    plan = api.PlanND(shape, batch, sign)
    y, z = plan.execute(x), plan.adjoint(x)
    for b in sorted({0, batch // 2, batch - 1}):
        for out, s in ((y, sign), (z, -sign)):
            ref = oracle.fftn(to_cpu(x[b:b + 1]).astype(np.complex128), len(shape), s, 1.0 if sign < 0 else 1.0 / n)
            assert per_transform_relerr(to_cpu(out[b]).reshape(1, -1), ref.reshape(1, -1)) <= TOL, (b, s)
