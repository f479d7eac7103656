"""The differentiable loss stores its gradient one way or another by size and
by whether a backward follows: the same loss and gradient, bit for bit, as the
plan's own call, at the sizes where that changes and in each mode."""
import pytest
import torch

from paper_2203_09384_amd import api
from gpu_util import need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,mib", [(64, 2), (64, 32), (64, 224), (2048, 2), (2048, 32), (2048, 256)])
@pytest.mark.parametrize("above", [0, 1])
def test_same_gradient(n, mib, above):
    need_gpu()
    batch = (mib << 17) // n + above
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.view_as_complex(torch.rand((batch, n, 2), generator=g, device="cuda").mul_(2).sub_(1))
    w = torch.rand((batch, n), generator=g, device="cuda")
    print(f"[case] n={n} batch={batch}", flush=True)
    loss, grad = api.get_plan(n, batch, -1).loss_grad(x, w)
    want = loss.sum()
    with torch.no_grad():
        assert torch.equal(api.weighted_power_loss(x, w), want)
    assert torch.equal(api.weighted_power_loss(x, w), want)  # x requires no gradient
    x.requires_grad_(True)
    got = api.weighted_power_loss(x, w)
    got.backward()
    assert torch.equal(got, want) and torch.equal(x.grad, grad)
