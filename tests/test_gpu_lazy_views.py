"""Lazily conjugated and negated tensors (x.conj(), torch._neg_view) as
inputs, gradients, weights and outputs: the transform of the values that the
tensor shows, on the first call of a shape as on later ones.  The same calls
on plain copies give the expected results, which are equal bit for bit (the
same kernels on the same values)."""
import pytest
import torch

from paper_2203_09384_amd import api
from gpu_util import need_gpu

pytestmark = pytest.mark.gpu
N, B = 64, 5


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


def real(*shape, seed=9):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.rand(shape, generator=g, device="cuda").mul_(2).sub_(1)


def signal(*shape, seed=9):
    return torch.view_as_complex(real(*shape, 2, seed=seed))


def plain(t):
    return t.resolve_conj().resolve_neg()


def lazy(t):
    """The values of t behind the conj bit (complex) or the neg bit (real)."""
    return t.conj().resolve_conj().conj() if t.is_complex() else torch._neg_view(-t)


def first_and_again(fn):
    """fn() with no plan cached, and twice more."""
    api._cache.clear()
    return [fn() for _ in range(3)]


CALLS = {
    "fft": (lambda x: api.fft(x), lambda: signal(B, N)),
    "ifft": (lambda x: api.ifft(x), lambda: signal(B, N)),
    "rfft": (lambda x: api.rfft(x), lambda: real(B, N)),
    "irfft": (lambda x: api.irfft(x), lambda: signal(B, N // 2 + 1)),
    "fft2": (lambda x: api.fft2(x), lambda: signal(B, 16, 8)),
    "fft_differentiable": (lambda x: api.fft_differentiable(x), lambda: signal(B, N)),
    "rfft_differentiable": (lambda x: api.rfft_differentiable(x), lambda: real(B, N)),
    "irfft_differentiable": (lambda x: api.irfft_differentiable(x), lambda: signal(B, N // 2 + 1)),
    "fftn_differentiable": (lambda x: api.fftn_differentiable(x, 2), lambda: signal(B, 16, 8)),
}


@pytest.mark.parametrize("name", CALLS)
def test_input(name):
    call, make = CALLS[name]
    x = make()
    want = call(x)
    assert lazy(x).is_conj() or lazy(x).is_neg()
    for got in first_and_again(lambda: call(lazy(x))):
        assert torch.equal(plain(got), plain(want))


@pytest.mark.parametrize("name", [c for c in CALLS if c.endswith("differentiable")])
def test_gradient(name):
    call, make = CALLS[name]
    x = make().requires_grad_(True)
    y = call(x)
    g = signal(*y.shape, seed=4) if y.is_complex() else real(*y.shape, seed=4)
    (want,) = torch.autograd.grad(call(x), x, g)

    def one():
        # the product's backward hands on a lazily conjugated gradient
        y = call(x)
        return torch.autograd.grad(y, x, lazy(g))[0]
    for got in first_and_again(one):
        assert torch.equal(plain(got), plain(want))


def test_gradient_through_conj():
    x = signal(B, N).requires_grad_(True)
    w = signal(B, N, seed=5)

    def one():
        y = api.fft_differentiable(x)
        return torch.autograd.grad((y.conj() * w).real.sum(), x)[0]
    first, again, _ = first_and_again(one)
    want = api.get_plan(N, B, -1).adjoint(w)  # d Re(conj(y) w) = w in dL/dRe + i dL/dIm
    assert torch.equal(plain(first), want) and torch.equal(plain(again), want)


@pytest.mark.parametrize("which", ["x", "w", "both"])
def test_loss(which):
    x, w = signal(B, N), real(B, N, seed=3)
    want = api.weighted_power_loss(x, w)
    xs, ws = (lazy(x) if which != "w" else x), (lazy(w) if which != "x" else w)
    for got in first_and_again(lambda: api.weighted_power_loss(xs, ws)):
        assert torch.equal(got, want)


@pytest.mark.parametrize("side", [None, "own"])
def test_plan(side):
    """execute and adjoint, on the current stream and on one given."""
    s = torch.cuda.Stream() if side else None
    x = signal(B, N)
    for plan in (api.Plan(N, B, -1), api.RaggedPlan([0, 64, 192, 320])):
        want, back = plan.execute(x), plan.adjoint(x)
        torch.cuda.synchronize()
        got, gback = plan.execute(lazy(x), stream=s), plan.adjoint(lazy(x), stream=s)
        store = torch.zeros_like(x)
        out = store.conj()
        assert plan.execute(lazy(x), out=out, stream=s) is out
        torch.cuda.synchronize()
        assert torch.equal(got, want) and torch.equal(gback, back)
        assert torch.equal(out.resolve_conj(), want) and torch.equal(store, want.conj().resolve_conj())


def test_plan_real_side():
    x = real(B, N)
    plan = api.Plan(N, B, -1, dtype="r32")
    want = plan.execute(x)
    assert torch.equal(plan.execute(lazy(x)), want)
    back = plan.adjoint(want)
    store = torch.zeros_like(x)
    out = torch._neg_view(store)
    plan.adjoint(lazy(want), out=out)
    assert torch.equal(out.resolve_neg(), back) and torch.equal(store, -back)


def test_loss_grad_and_scaled():
    x, w = signal(B, N), real(B, N, seed=3)
    plan = api.Plan(N, B, -1)
    loss, grad = plan.loss_grad(x, w)
    g = torch.zeros_like(x).conj()
    loss2, grad2 = plan.loss_grad(lazy(x), lazy(w), grad=g)
    assert grad2 is g and torch.equal(loss2, loss) and torch.equal(plain(g), grad)
    h = real(B, N, 2).half()
    half = api.Plan(N, B, -1, dtype="c16")
    want, exp = half.execute_scaled(h)
    got, exp2 = half.execute_scaled(lazy(h))
    assert torch.equal(got, want) and torch.equal(exp2, exp)


def test_refused_stays_refused():
    plan = api.Plan(N, B, -1)
    wide = signal(B, 2 * N)[:, ::2]
    for x in (wide, wide.conj()):
        with pytest.raises(ValueError):
            plan.execute(x)
    with pytest.raises(ValueError):
        plan.execute(signal(B, N), out=wide.conj())
    with pytest.raises(ValueError):
        plan.execute(signal(B, N).conj().cpu())
