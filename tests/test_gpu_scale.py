"""The kernel that scales the fused loss's gradient, called directly: odd and
even point counts from one, tensors on 8-byte boundaries, both kinds of store,
infinities and NaN.  Expected: torch's product of a complex tensor and a real
scalar (every operation is exact or correctly rounded in both)."""
import ctypes

import pytest
import torch

from paper_2203_09384_amd import native
from gpu_util import need_gpu

pytestmark = pytest.mark.gpu


def scale(x, f, out):
    fn = native.lib().mifft_scale_c32
    fn.argtypes = [ctypes.c_void_p] * 3 + [ctypes.c_int64, ctypes.c_void_p]
    fn.restype = ctypes.c_int
    return fn(x.data_ptr(), f.data_ptr(), out.data_ptr(), x.numel(), torch.cuda.current_stream().cuda_stream)


@pytest.mark.parametrize("points", [1, 2, 3, 511, 512, 513, 1025, 100001, (16 << 20) + 1, (16 << 20) + 2])
@pytest.mark.parametrize("offset", [0, 1])
def test_scale(points, offset):
    need_gpu()
    g = torch.Generator(device="cuda").manual_seed(points)
    x = torch.view_as_complex(torch.rand((points + offset, 2), generator=g, device="cuda").sub_(0.5))[offset:]
    if points > 2:
        x[1] = complex(float("inf"), 1.0)
        x[2] = complex(2.0, float("nan"))
    f = torch.full((1,), -1.75, device="cuda")
    out = torch.full((points + offset + 1,), 7 + 7j, dtype=torch.complex64, device="cuda")
    print(f"[case] scale points={points} offset={offset}", flush=True)
    assert scale(x, f, out[offset:offset + points]) == 0
    want = x * f
    got = torch.view_as_real(out[offset:offset + points])
    assert torch.equal(torch.nan_to_num(got, nan=123.0), torch.nan_to_num(torch.view_as_real(want), nan=123.0))
    assert out[-1] == 7 + 7j and (offset == 0 or out[0] == 7 + 7j)


def test_refuses_no_points():
    need_gpu()
    f = torch.ones(1, device="cuda")
    assert scale(torch.zeros(0, dtype=torch.complex64, device="cuda"), f, f) != 0
