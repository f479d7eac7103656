"""Kernel variants chosen by the size of the call: one call at each rule's
limit and one just above it, so that every choice runs in a plain plan, as
the last axis of a multidimensional one, and for real input.  Against the
FP64 oracle on sampled transforms; bar: relative L2 <= 1e-5."""
import numpy as np
import pytest
import torch

import oracle
from paper_2203_09384_amd import api
from gpu_util import need_gpu, per_transform_relerr, to_cpu

pytestmark = pytest.mark.gpu
TOL = 1e-5
C32 = [(8, 32), (9, 16), (10, 24), (10, 128), (11, 24), (12, 16), (13, 32)]
R32 = [(4, 32), (5, 32), (7, 24), (7, 96), (8, 24), (9, 32), (9, 192), (10, 24), (10, 96), (11, 32), (12, 32)]


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


def rand(*shape):
    g = torch.Generator(device="cuda").manual_seed(31)
    return torch.rand(shape, generator=g, device="cuda").mul_(2).sub_(1)


def sampled(batch):
    return torch.tensor(sorted({0, min(1, batch - 1), batch // 2, batch - 1}), device="cuda")


@pytest.mark.parametrize("log2n,mib", C32)
@pytest.mark.parametrize("above", [0, 1])
@pytest.mark.parametrize("sign", [-1, 1])
def test_complex(log2n, mib, above, sign):
    n = 1 << log2n
    batch = (mib << 17) // n + above
    x = torch.view_as_complex(rand(batch, n, 2))
    print(f"[case] n={n} batch={batch} sign={sign}", flush=True)
    y = api.Plan(n, batch, sign).execute(x)
    at = sampled(batch)
    xs = to_cpu(x[at]).astype(np.complex128)
    assert per_transform_relerr(to_cpu(y[at]), oracle.forward(xs) if sign < 0 else oracle.inverse(xs)) <= TOL
    # pairs of transforms as arrays of 2 x n
    if batch % 2 == 0:
        y2 = api.PlanND((2, n), batch // 2, -1).execute(x)
        k = sampled(batch // 2)
        ref = oracle.fftn(to_cpu(x.view(-1, 2, n)[k]).astype(np.complex128), 2)
        assert per_transform_relerr(to_cpu(y2.view(-1, 2 * n)[k]), ref.reshape(len(k), -1)) <= TOL


@pytest.mark.parametrize("log2m,mib", R32)
@pytest.mark.parametrize("above", [0, 1])
def test_real(log2m, mib, above):
    n = 2 << log2m
    batch = (mib << 18) // n + above
    x = rand(batch, n)
    print(f"[case] real n={n} batch={batch}", flush=True)
    X = api.Plan(n, batch, -1, dtype="r32").execute(x)
    back = api.Plan(n, batch, +1, dtype="r32").execute(X)
    at = sampled(batch)
    assert per_transform_relerr(to_cpu(X[at]), oracle.rfft(to_cpu(x[at]).astype(np.float64))) <= TOL
    assert per_transform_relerr(to_cpu(back[at]), to_cpu(x[at])) <= 2 * TOL
