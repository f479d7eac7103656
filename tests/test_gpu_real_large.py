"""Real input above 2^15, whose split is folded into the four-step passes:
every length, batches that fill the XCD dealing of row tiles or not, all four
maps (R2C, C2R and their adjoints), and batches of several chunks.  Against
the FP64 oracle; bar, as for every FP32 transform: relative L2 <= 1e-5."""
import numpy as np
import pytest
import torch

import oracle
from paper_2203_09384_amd import api, synth
from gpu_util import need_gpu, per_transform_relerr, to_cpu, to_gpu

pytestmark = pytest.mark.gpu
TOL = 1e-5


@pytest.mark.parametrize("L", range(16, 22))
@pytest.mark.parametrize("batch", [1, 8, 11])
def test_all_maps(L, batch):
    if batch > 1 and L > 19:
        batch = 3 if batch == 8 else 9
    n = 1 << L
    x = synth.uniform_real(83, (batch, n), key=(L,))
    X = synth.uniform_complex(83, (batch, n // 2 + 1), key=(L, 1))
    print(f"[case] real n={n} batch={batch}", flush=True)
    fwd, inv = api.Plan(n, batch, -1, dtype="r32"), api.Plan(n, batch, +1, dtype="r32")
    x64, X64 = x.astype(np.float64), X.astype(np.complex128)
    for got, want in ((fwd.execute(to_gpu(x)), oracle.rfft(x64)), (inv.execute(to_gpu(X)), oracle.irfft(X64, n)),
                      (fwd.adjoint(to_gpu(X)), oracle.rfft_adjoint(X64, n)),
                      (inv.adjoint(to_gpu(x)), oracle.irfft_adjoint(x64))):
        assert per_transform_relerr(to_cpu(got), want) <= TOL


@pytest.mark.parametrize("L", [16, 18, 21])
def test_chunks(L):
    """One chunk of 128 MiB and a short second one, which shares the first
    one's workspace."""
    n = 1 << L
    per = (128 << 20) // (4 * n)
    batch = per + 3
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.rand((batch, n), generator=g, device="cuda").mul_(2).sub_(1)
    print(f"[case] real chunks n={n} batch={batch}", flush=True)
    X = api.Plan(n, batch, -1, dtype="r32").execute(x)
    back = api.Plan(n, batch, +1, dtype="r32").execute(X)
    at = torch.tensor([0, per - 1, per, batch - 1], device="cuda")
    assert per_transform_relerr(to_cpu(X[at]), oracle.rfft(to_cpu(x[at]).astype(np.float64))) <= TOL
    assert per_transform_relerr(to_cpu(back[at]), to_cpu(x[at])) <= 2 * TOL
