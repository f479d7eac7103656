"""Transforms on both sides of every size at which the kernel variant
changes, the sizes taken from the query itself, against the FP64 oracle on
sampled transforms; bar, as for every FP32 transform: relative L2 <= 1e-5."""
import numpy as np
import pytest
import torch

import oracle
from paper_2203_09384_amd import api
from gpu_util import need_gpu, per_transform_relerr, to_cpu

pytestmark = pytest.mark.gpu
TOL = 1e-5


def switches(n, sign, dtype, elem):
    """Batches up to 256 MiB at which the next larger one runs another variant."""
    def of(batch):
        d = api.query(n, batch, sign, dtype)
        return d["ept"], d["wg"], d["variant"]
    got = []
    for mib in range(1, 256):
        batch = (mib << 20) // (n * elem)
        if of(batch) != of(batch + 1):
            got.append(batch)
    return got


@pytest.mark.parametrize("n", [256, 512, 1024, 2048, 4096, 8192])
@pytest.mark.parametrize("sign", [-1, 1])
def test_complex(n, sign):
    need_gpu()
    g = torch.Generator(device="cuda").manual_seed(33)
    found = switches(n, sign, "c32", 8)
    assert found
    for batch in [b + d for b in found for d in (0, 1)]:
        x = torch.view_as_complex(torch.rand((batch, n, 2), generator=g, device="cuda").mul_(2).sub_(1))
        print(f"[case] n={n} batch={batch} sign={sign}", flush=True)
        y = api.Plan(n, batch, sign).execute(x)
        at = torch.tensor([0, batch // 2, batch - 1], device="cuda")
        xs = to_cpu(x[at]).astype(np.complex128)
        assert per_transform_relerr(to_cpu(y[at]), oracle.forward(xs) if sign < 0 else oracle.inverse(xs)) <= TOL


@pytest.mark.parametrize("n", [32, 64, 256, 512, 1024, 2048, 4096, 8192])
@pytest.mark.parametrize("sign", [-1, 1])
def test_real(n, sign):
    """A plan of `sign`: its own direction and its adjoint."""
    need_gpu()
    g = torch.Generator(device="cuda").manual_seed(34)
    found = switches(n, sign, "r32", 4)
    assert found
    for batch in [b + d for b in found for d in (0, 1)]:
        x = torch.rand((batch, n), generator=g, device="cuda").mul_(2).sub_(1)
        print(f"[case] real n={n} batch={batch} sign={sign}", flush=True)
        plan = api.Plan(n, batch, sign, dtype="r32")
        at = torch.tensor([0, batch // 2, batch - 1], device="cuda")
        bins = oracle.rfft(to_cpu(x[at]).astype(np.float64))
        if sign < 0:
            X = plan.execute(x)
            assert per_transform_relerr(to_cpu(X[at]), bins) <= TOL
            continue
        # adjoint of the inverse: the bins over n, interior ones doubled
        X = plan.adjoint(x)
        weight = np.full(n // 2 + 1, 2.0 / n)
        weight[[0, -1]] = 1.0 / n
        assert per_transform_relerr(to_cpu(X[at]), bins * weight) <= TOL
        back = plan.execute(api.Plan(n, batch, -1, dtype="r32").execute(x))
        assert per_transform_relerr(to_cpu(back[at]), to_cpu(x[at])) <= 2 * TOL
