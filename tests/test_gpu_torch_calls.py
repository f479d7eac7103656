"""The C++ calls on torch tensors against the Python autograd functions that
they stand in for: the same kernels on the same inputs, so equal bit for
bit; and calls outside the ordinary case, which go the Python way."""
import gc

import pytest
import torch

from paper_2203_09384_amd import api
from paper_2203_09384_amd.native import MifftError
from gpu_util import need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


def rand(*shape, real=False):
    x = torch.rand(shape if real else shape + (2,), device="cuda") * 2 - 1
    return x if real else torch.view_as_complex(x)


CASES = {
    "fft": (lambda x: api.fft_differentiable(x), lambda x: api.FFTFn.apply(x, -1), lambda: rand(3, 5, 64)),
    "ifft": (lambda x: api.fft_differentiable(x, +1), lambda x: api.FFTFn.apply(x, +1), lambda: rand(7, 4096)),
    "rfft": (lambda x: api.rfft_differentiable(x), lambda x: api.RFFTFn.apply(x), lambda: rand(5, 128, real=True)),
    "irfft": (lambda x: api.irfft_differentiable(x), lambda x: api.IRFFTFn.apply(x, 128), lambda: rand(5, 65)),
    "fft2": (lambda x: api.fftn_differentiable(x, 2), lambda x: api.FFTNFn.apply(x, 2, -1), lambda: rand(3, 16, 32)),
}


@pytest.mark.parametrize("name", CASES)
def test_linear_maps(name):
    call, reference, make = CASES[name]
    x = make().requires_grad_(True)
    want = reference(x)  # also makes the cached plan
    g = torch.randn_like(want)
    (gw,) = torch.autograd.grad(want, x, g)
    y = call(x)
    assert type(y.grad_fn).__name__ != type(want.grad_fn).__name__  # the C++ function ran
    (gy,) = torch.autograd.grad(y, x, g, retain_graph=True)
    (again,) = torch.autograd.grad(y, x, g)
    assert torch.equal(y, want) and torch.equal(gy, gw) and torch.equal(again, gw)
    assert torch.equal(call(x.detach()), want)


def test_loss():
    x, w = rand(9, 256).requires_grad_(True), torch.rand(9, 256, device="cuda")
    want = api.WeightedPowerLossFn.apply(x, w, -1)
    (gw,) = torch.autograd.grad(want * 3, x)
    loss = api.weighted_power_loss(x, w)
    (g,) = torch.autograd.grad(loss * 3, x)
    assert torch.equal(loss, want) and torch.equal(g, gw)


def test_functions_and_plans():
    x, r = rand(6, 512), rand(6, 512, real=True)
    X = api.rfft(r)
    for f in (lambda: api.fft(x), lambda: api.ifft(x), lambda: api.rfft(r), lambda: api.irfft(X),
              lambda: api.fftn(x.view(6, 16, 32), 2)):
        assert torch.equal(f(), f())
    for p, a in ((api.Plan(512, 6, -1), x), (api.Plan(512, 6, +1, dtype="r32"), X), (api.RaggedPlan([0, 2048, 3072]), x)):
        y, s = p.execute(a), torch.cuda.current_stream()
        assert torch.equal(y, p.execute(a, out=torch.empty_like(y))) and torch.equal(y, p.execute(a, stream=s))
        assert torch.equal(p.adjoint(y), p.adjoint(y, stream=s))
    h = api.Plan(64, 3, -1, dtype="c16")
    a = torch.randn(3, 64, 2, device="cuda").half()
    assert torch.equal(h.execute(a), h.execute(a, stream=torch.cuda.current_stream()))
    for got, want in zip(h.execute_scaled(a), h.execute_scaled(a, stream=torch.cuda.current_stream())):
        assert torch.equal(got, want)


def test_outside_the_ordinary_case():
    x = rand(8, 64)
    want = api.fft(x)
    assert torch.equal(api.fft(x.t().contiguous().t()), want)  # strided

    class Sub(torch.Tensor):
        pass

    assert torch.equal(api.fft(x.as_subclass(Sub)).as_subclass(torch.Tensor), want)
    p = api.Plan(64, 8, -1)
    for bad in (x[:7], x.to(torch.complex128), x.cpu(), x.t()):
        with pytest.raises(ValueError):
            p.execute(bad)
    with pytest.raises(ValueError):
        p.execute(x, out=torch.empty_like(x)[:7])
    with pytest.raises(RuntimeError):
        torch.func.vmap(api.fft_differentiable)(x)
    with pytest.raises((RuntimeError, NotImplementedError)):
        torch.func.jvp(api.fft_differentiable, (x,), (x,))
    with pytest.raises(MifftError):
        p.execute(x, out=x)  # overlap


def test_saved_tensor_hooks_see_the_loss_gradient():
    x, w = rand(4, 64).requires_grad_(True), torch.rand(4, 64, device="cuda")
    api.weighted_power_loss(x, w)
    seen = []
    with torch.autograd.graph.saved_tensors_hooks(lambda t: (seen.append(t.shape), t)[1], lambda t: t):
        loss = api.weighted_power_loss(x, w)
    assert seen == [x.shape]
    torch.autograd.grad(loss, x)


def test_graph_outlives_its_plan_object():
    x = rand(4, 32).requires_grad_(True)
    key = (0, 32, 4, -1, "c32")
    want = api.FFTFn.apply(x, -1)
    y = api.fft_differentiable(x)
    g = torch.randn_like(y)
    (gw,) = torch.autograd.grad(want, x, g)
    del want
    api._cache.pop(key)
    gc.collect()
    (gy,) = torch.autograd.grad(y, x, g)
    assert torch.equal(gy, gw)


def test_closed_plan_is_refused():
    p = api.Plan(64, 8, -1)
    p.close()
    with pytest.raises(MifftError):
        p.execute(rand(8, 64))


@pytest.mark.parametrize("batch,n", [(1, 2), (1, 4), (3, 64), (16385, 2048)])
@pytest.mark.parametrize("factor", [1.0, -2.5, float("inf"), float("nan")])
def test_loss_backward_scales_like_torch(batch, n, factor):
    """The scaling kernel against torch's product, at odd and even point
    counts, above the size at which it streams, and for factors that are not
    finite: bit for bit."""
    x = rand(batch, n).requires_grad_(True)
    w = torch.rand(batch, n, device="cuda")
    f = torch.tensor(factor, device="cuda")
    api.weighted_power_loss(x, w)
    loss = api.weighted_power_loss(x, w)
    _, unit = api.get_plan(n, batch, -1, "c32", 0).loss_grad(x.detach(), w)
    (got,) = torch.autograd.grad(loss, x, f)
    want = unit * f
    assert torch.equal(torch.view_as_real(got).view(torch.int32) if factor == factor else torch.view_as_real(got).isnan(),
                       torch.view_as_real(want).view(torch.int32) if factor == factor else torch.view_as_real(want).isnan())


def test_loss_gradient_of_gradient_and_batched():
    """A backward that is itself differentiated, or run under vmap, keeps
    torch's own product."""
    x, w = rand(4, 64).requires_grad_(True), torch.rand(4, 64, device="cuda")
    api.weighted_power_loss(x, w)
    g = torch.tensor(2.0, device="cuda", requires_grad=True)
    (grad,) = torch.autograd.grad(api.weighted_power_loss(x, w), x, g, create_graph=True)
    (gg,) = torch.autograd.grad(grad.real.sum(), g)
    assert torch.allclose(gg, grad.real.sum() / 2)
    several = torch.autograd.grad(api.weighted_power_loss(x, w), x, torch.tensor([1.0, 3.0], device="cuda"),
                                  is_grads_batched=True)[0]
    assert torch.equal(several[1], 3 * several[0])
