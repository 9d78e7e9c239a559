"""The dense convolution's tiles (csrc/alcs_dense.hip) at the sizes where they can go wrong, against the
oracle: channels that are no multiple of a step, channel and pixel tiles with a remainder, tiles over
several images, every number of staged positions per thread, 3x3 tiles of 64 pixels, and the layers
that fall to the word-by-word kernel, on 64 and on 128 channels."""
import numpy as np
import pytest

import workloads
from gpu_util import TOL, oracle_ref, rel_err, run_dense

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,stride,Cin,Cout,H,W,N", [
    (3, 1, 8, 32, 12, 11, 1),      # one step of 8 channels
    (3, 1, 9, 31, 4, 4, 40),       # a step and a channel; 8 images in a tile
    (3, 1, 24, 33, 1, 1, 300),     # one-pixel images: 128 are past the staging, tiles of 64
    (3, 1, 16, 65, 3, 2, 25),      # 21 images in a tile
    (3, 2, 17, 130, 15, 9, 5),
    (3, 2, 12, 40, 33, 58, 3),     # more than 512 staged positions
    (3, 1, 10, 70, 13, 140, 2),    # 768 to 1024 of them
    (3, 1, 5, 20, 3, 300, 2),      # wider than the staging
    (3, 2, 3, 32, 40, 224, 2),
    (3, 2, 20, 70, 112, 112, 2),   # tiles of 64 pixels, 904 positions, over the seam of two images
    (3, 2, 9, 33, 105, 157, 1),    # 795
    (3, 2, 13, 40, 31, 146, 1),    # 735: three a thread
    (3, 2, 8, 64, 64, 203, 1),     # the widest image
    (3, 2, 12, 64, 112, 112, 21),  # few input channels on many tiles: word by word, 64 channels
    (3, 2, 17, 120, 112, 112, 21),  # 128 channels
    (1, 1, 16, 16, 5, 3, 9),       # one step of 16 channels
    (1, 1, 32, 16, 5, 3, 9),       # two
    (1, 1, 8, 40, 6, 5, 4),        # half of one
    (1, 1, 31, 64, 1, 1, 70),
    (1, 1, 97, 129, 9, 7, 31),
    (1, 2, 64, 30, 31, 17, 6),
    (1, 1, 160, 200, 56, 56, 5),   # several tiles a compute unit
    (3, 1, 64, 256, 30, 30, 12),   # 128 x 128
    # split operands: 128 x 256 with and without remainders, 128 x 128, 64 x 128, one step, a step and a channel,
    # more than 512 positions (float32 again)
    (3, 1, 16, 128, 28, 28, 64), (3, 1, 9, 130, 27, 29, 70), (3, 1, 17, 250, 14, 14, 130),
    (3, 1, 8, 736, 28, 28, 9), (3, 1, 13, 715, 14, 11, 10), (3, 1, 5, 330, 28, 28, 6), (3, 1, 24, 780, 7, 7, 70),
    (3, 2, 12, 300, 30, 26, 40), (3, 1, 8, 400, 6, 90, 30),
    (1, 1, 300, 256, 28, 28, 64), (1, 1, 320, 250, 27, 29, 64), (1, 2, 333, 512, 56, 55, 60),   # 1x1, 128 x 256
    (1, 1, 1001, 250, 14, 14, 64), (1, 1, 992, 255, 13, 15, 64), (1, 1, 993, 256, 1, 1, 20000),  # 128 x 128, and images of one pixel
])
def test_dense_tiles(k, stride, Cin, Cout, H, W, N):
    L = workloads.Layer("tile", Cin, Cout, H, W, k=k, stride=stride, N=N, V=1, sparsity=0.0, w_std=0.1,
                        mask_kind="none")
    d = workloads.make_layer(L, 8800 + Cin + Cout, with_bias=True)
    got = run_dense(d)
    assert not np.isnan(got).any()
    assert rel_err(got, oracle_ref(d)) <= TOL


def test_split_operands_with_infinities():
    """Where one input is infinite the outputs that see it are, and all others are what they were; the largest finite
    input stays finite."""
    import torch

    import paper_2109_00170_amd as alcs
    g = torch.Generator().manual_seed(6)
    X = torch.rand((64, 16, 28, 28), generator=g).cuda()
    F = (0.1 + torch.rand((128, 16, 3, 3), generator=g)).cuda() * 0.01
    Y = [torch.empty((64, 128, 28, 28), device="cuda") for _ in range(3)]
    alcs.alcs_dense_conv(F, X, None, Y[0])
    want = torch.nn.functional.conv2d(X.cpu().double(), F.cpu().double(), padding=1)
    assert float((Y[0].cpu() - want).abs().max() / want.abs().max()) <= TOL
    for big, y in ((float("inf"), Y[1]), (3.4e38, Y[2])):
        Z = X.clone()
        Z[5, 3, 10, 27] = big
        alcs.alcs_dense_conv(F, Z, None, y)
        sees = torch.zeros(Y[0].shape, dtype=torch.bool, device="cuda")
        sees[5, :, 9:12, 26:28] = True
        assert torch.equal(y[~sees], Y[0][~sees])
        got = y[sees].cpu()
        if big == float("inf"):
            assert bool((got == big).all())
        else:
            assert bool(torch.isfinite(got).all()) and float(got.min()) > 1e35


def test_dense_tile_beyond_2_31_bytes():
    """A tile whose input spans more than 2^31 bytes: 17 images of 4x4 with 3e6 channels, nearly all zero."""
    import torch

    import paper_2109_00170_amd as alcs
    C, N = 3_000_000, 17
    some = torch.cat([torch.arange(50), torch.arange(1_500_001, 1_500_050), torch.arange(C - 53, C)])
    g = torch.Generator().manual_seed(5)
    x = torch.randn((N, len(some), 4, 4), generator=g)
    X = torch.zeros((N, C, 4, 4), device="cuda")
    X[:, some.cuda()] = x.cuda()
    F = torch.randn((3, C, 1, 1), generator=g)
    Y = torch.full((N, 3, 2, 2), float("nan"), device="cuda")
    alcs.alcs_dense_conv(F.cuda(), X, None, Y, stride=2)
    want = torch.nn.functional.conv2d(x.double(), F[:, some].double(), stride=2).numpy()
    assert rel_err(Y.cpu().numpy(), want) <= TOL
