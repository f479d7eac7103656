"""Transforms of several passes over batches large enough to run chunk by
chunk: transforms at both ends of a chunk and in a short last one, against
the FP64 oracle.  Bar, as for every FP32 transform: relative L2 <= 1e-5."""
import numpy as np
import pytest
import torch

import oracle
from paper_2203_09384_amd import api
from gpu_util import need_gpu, per_transform_relerr, to_cpu

pytestmark = pytest.mark.gpu
TOL = 1e-5
CHUNK = 256 << 20  # bytes


def signal(*shape):
    g = torch.Generator(device="cuda").manual_seed(77)
    return torch.view_as_complex(torch.rand(shape + (2,), generator=g, device="cuda").mul_(2).sub_(1))


@pytest.mark.parametrize("L", [15, 16, 17, 18, 20])
@pytest.mark.parametrize("sign", [-1, 1])
def test_four_step_chunks(L, sign):
    n = 1 << L
    per = CHUNK // (8 * n)
    batch = per + 3
    x = signal(batch, n)
    print(f"[case] four-step chunks n={n} batch={batch} sign={sign}", flush=True)
    y = api.Plan(n, batch, sign).execute(x)
    at = torch.tensor([0, per - 1, per, batch - 1], device="cuda")
    xs = to_cpu(x[at]).astype(np.complex128)
    assert per_transform_relerr(to_cpu(y[at]), oracle.forward(xs) if sign < 0 else oracle.inverse(xs)) <= TOL


@pytest.mark.parametrize("shape,batch", [((512, 1024), 67), ((64, 128, 128), 17), ((64, 512, 1024), 1),
                                         ((256, 512, 512), 1), ((4, 32768), 258)], ids=str)
@pytest.mark.parametrize("sign", [-1, 1])
def test_nd_chunks(shape, batch, sign):
    """Chunks of whole arrays, and of planes where one array exceeds a chunk
    (256 x 512 x 512: 512 MiB)."""
    n = int(np.prod(shape))
    x = signal(batch, *shape)
    print(f"[case] nd chunks shape={shape} batch={batch} sign={sign}", flush=True)
    y = api.PlanND(shape, batch, sign).execute(x)
    for b in {0, batch - 1}:
        ref = oracle.fftn(to_cpu(x[b:b + 1]).astype(np.complex128), len(shape), sign, 1.0 if sign < 0 else 1.0 / n)
        assert per_transform_relerr(to_cpu(y[b]).reshape(1, -1), ref.reshape(1, -1)) <= TOL


@pytest.mark.parametrize("shape", [(4, 4), (8, 8), (16, 16), (64, 64), (128, 128), (8, 8, 8), (16, 16, 16), (4, 8, 64)],
                         ids=str)
@pytest.mark.parametrize("sign", [-1, 1])
def test_single_pass_nd_beyond_the_cache(shape, sign):
    """Single-pass 2D / 3D transforms whose output exceeds 256 MiB."""
    n = int(np.prod(shape))
    batch = (257 << 17) // n + 1
    x = signal(batch, *shape)
    print(f"[case] nd beyond the cache shape={shape} batch={batch} sign={sign}", flush=True)
    y = api.PlanND(shape, batch, sign).execute(x)
    at = torch.tensor([0, 1, batch // 2, batch - 1], device="cuda")
    ref = oracle.fftn(to_cpu(x[at]).astype(np.complex128), len(shape), sign, 1.0 if sign < 0 else 1.0 / n)
    assert per_transform_relerr(to_cpu(y[at]).reshape(4, -1), ref.reshape(4, -1)) <= TOL
