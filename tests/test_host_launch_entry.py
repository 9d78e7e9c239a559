"""The native entry of the launches turns what PyTorch throws, integers that do not fit, and tensors a kernel
would read beyond, into Python errors."""
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


@pytest.mark.gpu
def test_dimensions_that_do_not_fit_are_refused():
    n = 2 ** 32 + 1   # cut to 32 bits: one image
    W, X, Y = (torch.zeros(shape, device="cuda") for shape in ((0, 0, 1, 1), (n, 0, 1, 1), (n, 0, 1, 1)))
    with pytest.raises(ValueError, match="dimension"):
        alcs.alcs_dense_conv(W, X, None, Y)


@pytest.mark.gpu
@pytest.mark.parametrize("kh,kw", [(3, 1), (1, 3)])
def test_filters_that_are_not_square_are_refused(kh, kw):
    W, X = torch.zeros((8, 4, kh, kw), device="cuda"), torch.zeros((1, 4, 5, 5), device="cuda")
    mask = torch.ones((2, 4, kh, kh), dtype=torch.uint8, device="cuda")
    for call in (lambda: alcs.alcs_dense_conv(W, X, None, torch.zeros((1, 8, 5, 5), device="cuda")),
                 lambda: alcs.alcs_block_scores(W, 4),
                 lambda: alcs.alcs_block_scores(W, 4, scores=torch.zeros((2, 4, kh, kh), device="cuda")),
                 lambda: alcs.alcs_pack_network_device([W], [mask], 4),
                 lambda: alcs.alcs_pack_workspace_bytes([W], [mask], 4),
                 lambda: alcs.alcs_pack_weights_device(W, mask, 4),
                 lambda: alcs.alcs_pack_csr_device(W, mask, 4)):
        with pytest.raises(ValueError):
            call()


@pytest.mark.gpu
def test_bias_shorter_than_the_channels_is_refused():
    X, Y = torch.ones((1, 4, 5, 5), device="cuda"), torch.zeros((1, 8, 5, 5), device="cuda")
    W, D, Z = torch.ones((8, 4, 1, 1), device="cuda"), torch.ones((4, 3, 3), device="cuda"), torch.zeros_like(X)
    p = alcs.alcs_pack_weights_device(W, None, 4)
    bf = [t.to(torch.bfloat16) for t in (X, Y)]
    p.add_bf16_weights()
    b8, b4 = torch.zeros(8, device="cuda"), torch.zeros(4, device="cuda")

    def calls(b8, b4):
        yield lambda: alcs.alcs_sparse_conv(p, X, b8, Y)
        yield lambda: alcs.alcs_sparse_conv_fused(p, X, b8, None, Y)
        yield lambda: alcs.alcs_sparse_conv_bf16(p, bf[0], b8, None, bf[1])
        yield lambda: alcs.alcs_sparse_conv_bf16_mfma(p, bf[0], b8, None, bf[1])
        yield lambda: alcs.alcs_dense_conv(W, X, b8, Y)
        yield lambda: alcs.alcs_depthwise_conv(D, X, b4, Z)
        yield lambda: alcs.alcs_dw_sparse_conv_fused(p, D, None, X, b8, None, Y)
        yield lambda: alcs.alcs_dw_sparse_conv_fused(p, D, b4, X, None, None, Y)

    for call in calls(b8, b4):
        call()
    for call in calls(torch.zeros((1, 9, 1, 1), device="cuda"), torch.zeros(5, device="cuda")):  # more than needed
        call()
    for call in calls(b8[:7], b4[:3]):
        with pytest.raises(ValueError, match="entries"):
            call()
