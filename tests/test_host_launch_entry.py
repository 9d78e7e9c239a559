"""The native entry of the launches turns what PyTorch throws, and integers that do not fit, into Python errors."""
import pytest
import torch
from torch._subclasses.fake_tensor import FakeTensorMode

import paper_2109_00170_amd as alcs


def test_tensors_without_storage_are_refused():
    # a tracer's tensors claim to be on the GPU and throw when their address is asked for
    with FakeTensorMode():
        W, X, Y = (torch.empty((4, 4, 1, 1), device="cuda") for _ in range(3))
    with pytest.raises(RuntimeError):
        alcs.alcs_dense_conv(W, X, None, Y)


@pytest.mark.gpu
@pytest.mark.parametrize("stride", [2 ** 32 + 1, 2 ** 64 + 1])
def test_strides_that_do_not_fit_are_refused(stride):
    # cut to 32 bits they would read as 1
    W, X, Y = (torch.zeros((4, 4, 1, 1), device="cuda") for _ in range(3))
    with pytest.raises((ValueError, OverflowError)):
        alcs.alcs_dense_conv(W, X, None, Y, stride=stride)
