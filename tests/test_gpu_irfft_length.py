"""irfft's length argument: lengths that do not belong to the given bins are
refused, also where a plan that would fit the tensor is already cached."""
import pytest
import torch

from paper_2203_09384_amd import api
from paper_2203_09384_amd.native import MifftError
from gpu_util import need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


@pytest.mark.parametrize("call", [api.irfft, api.irfft_differentiable], ids=["irfft", "irfft_differentiable"])
@pytest.mark.parametrize("n", [0, -1, -2, -4, 3, 4])
def test_wrong_length(call, n):
    X = torch.zeros(3, 2, dtype=torch.complex64, device="cuda")  # 2 bins: n = 2
    assert call(X).shape == (3, 2)
    assert call(X, 2).shape == (3, 2)  # its plan is cached now
    with pytest.raises((ValueError, MifftError, ZeroDivisionError)):
        call(X, n)
