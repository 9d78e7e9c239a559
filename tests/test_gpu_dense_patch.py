"""The dense convolution's tiles (csrc/alcs_dense.hip) at the sizes where they can go wrong, against the
oracle: channels that are no multiple of a step, channel and pixel tiles with a remainder, tiles over
several images, 3x3 tiles of 64 pixels, and the layers that fall to the word-by-word kernel, on 64 and on
128 channels.  Shapes of fewer than 256 tiles of 32 x 32 outputs that do not run on split operands are k_dense_few's now: they keep
their places as its ragged cases, and test_gpu_dense_few.py has larger launches of the tiles they stood for.  That every kernel the
library can choose is among the shapes of the two files is checked without a GPU (test_host_dense_plan.py)."""
import numpy as np
import pytest

import workloads
from dense_plan import dense_plan
from gpu_util import TOL, oracle_ref, rel_err, run_dense

pytestmark = pytest.mark.gpu


TILES = [
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
    (3, 1, 64, 256, 30, 30, 12),
    # around split operands and float32: one step, a step and a channel, channel and pixel tiles with and without
    # remainders, about 512 positions
    (3, 1, 16, 128, 28, 28, 64), (3, 1, 9, 130, 27, 29, 70), (3, 1, 17, 250, 14, 14, 130),
    (3, 1, 8, 736, 28, 28, 9), (3, 1, 13, 715, 14, 11, 10), (3, 1, 5, 330, 28, 28, 6), (3, 1, 24, 780, 7, 7, 70),
    (3, 2, 12, 300, 30, 26, 40), (3, 1, 8, 400, 6, 90, 30),
    (1, 1, 300, 256, 28, 28, 64), (1, 1, 320, 250, 27, 29, 64), (1, 2, 333, 512, 56, 55, 60),   # 1x1, 128 x 256
    (1, 1, 1001, 250, 14, 14, 64), (1, 1, 992, 255, 13, 15, 64), (1, 1, 993, 256, 1, 1, 20000),  # 128 x 128, and images of one pixel
    # tiles that none of these takes
    (1, 2, 10, 9, 10, 30, 219),                             # 1x1, 32 x 128
    (3, 2, 73, 204, 13, 52, 82), (3, 2, 41, 94, 11, 99, 77),   # float32, 128 x 128: 742 and 1010 positions
    (3, 2, 33, 105, 55, 33, 59), (3, 2, 13, 71, 71, 84, 19),   # split, 64 x 128: 700 and 1020
    (3, 1, 10, 33, 40, 8, 166),                             # float32, 64 x 128
    (3, 1, 133, 39, 81, 57, 4), (3, 2, 10, 35, 12, 57, 95),   # split, 64 x 128: 472 and 826 positions
    (3, 1, 9, 118, 19, 70, 19), (3, 1, 20, 419, 25, 72, 4),   # split, 128 x 128: 504 and 518
    (3, 1, 9, 97, 16, 20, 130),                             # split, 128 x 256
]


@pytest.mark.parametrize("k,stride,Cin,Cout,H,W,N", TILES)
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


# (k, stride, Cin, Cout, H, W, N) of each tile on split operands: 128 x 256, 128 x 128 and 64 x 128 for 3x3 (these with
# one and two staged positions per thread), 128 x 256 and 128 x 128 for 1x1; steps of 8 (32) channels and a remainder.
SPLIT = [(3, 1, 17, 250, 14, 14, 130), (3, 1, 9, 118, 19, 70, 19), (3, 1, 20, 419, 25, 72, 4), (3, 1, 133, 39, 81, 57, 4),
         (3, 2, 10, 35, 12, 57, 95), (1, 1, 320, 250, 27, 29, 64), (1, 1, 1001, 250, 14, 14, 64)]


@pytest.fixture(autouse=True)
def split_tiles(request):
    """The tests that name SPLIT shapes run on split operands on this GPU too."""
    import torch
    if request.node.originalname not in ("test_dense_tiles", "test_split_operands_with_infinities", "test_dense_tile_beyond_2_31_bytes"):
        v = request.node.callspec.params
        cus = torch.cuda.get_device_properties(0).multi_processor_count
        assert dense_plan(*(v[n] for n in ("k", "stride", "Cin", "Cout", "H", "W", "N")), cus=cus)[0][1] == "split"


def dense64(X, F, stride):
    import torch
    k = F.shape[-1]
    return torch.nn.functional.conv2d(X.cpu().double(), F.cpu().double(), stride=stride, padding=k // 2)


def dense_gpu(X, F, stride, like):
    import torch

    import paper_2109_00170_amd as alcs
    Y = torch.full(like.shape, float("nan"), device="cuda")
    alcs.alcs_dense_conv(F.cuda(), X.cuda(), None, Y, stride=stride)
    return Y.cpu()


@pytest.mark.parametrize("k,stride,Cin,Cout,H,W,N", SPLIT)
def test_one_term_is_one_rounding(k, stride, Cin, Cout, H, W, N):
    """Filters of one weight, another channel and tap for each output: the result is the rounded product, as of one
    multiply-add in float32 (2^-24 relative).  Leaving out any of the eight products of the operands' parts is 2^-22 or more on
    some outputs; what is left out is 2^-30, and the sum of the smaller products adds roundings of 2^-31 each."""
    import torch
    g = torch.Generator().manual_seed(Cin)
    X = torch.randn((N, Cin, H, W), generator=g)
    F = torch.zeros((Cout, Cin, k, k))
    o = torch.arange(Cout)
    F.view(Cout, Cin, k * k)[o, o * 7 % Cin, o % (k * k)] = torch.randn(Cout, generator=g)
    want = dense64(X, F, stride)
    got = dense_gpu(X, F, stride, want)
    assert float(((got - want).abs() - want.abs() * (2.0 ** -24 * (1 + 2.0 ** -3))).max()) <= 0


@pytest.mark.parametrize("k,stride,Cin,Cout,H,W,N", SPLIT)
def test_split_sums_are_float32_sums(k, stride, Cin, Cout, H, W, N):
    """Error of whole layers: one rounding (2^-25 of the running sum in the mean) per 16 rows of K in the large sum, and
    the seven smaller ones in sums 2^-7 of its size."""
    import torch
    g = torch.Generator().manual_seed(Cin + 1)
    X, F = torch.randn((N, Cin, H, W), generator=g), torch.randn((Cout, Cin, k, k), generator=g)
    want = dense64(X, F, stride)
    got = dense_gpu(X, F, stride, want)
    steps = -(-Cin * k * k // 16) + 2
    assert float((got - want).norm() / want.norm()) <= 2.0 ** -24 * steps ** 0.5


@pytest.mark.parametrize("k,stride,Cin,Cout,H,W,N", [SPLIT[0], SPLIT[1], SPLIT[4], SPLIT[5], SPLIT[6]])
@pytest.mark.parametrize("size", [2e-31, 1e-33, 1e-35, 4e-37])
@pytest.mark.parametrize("which", ["input", "weights"])
def test_small_operands_keep_their_bits(k, stride, Cin, Cout, H, W, N, size, which):
    """Numbers whose lowest bits lie below the smallest bfloat16 number, in one image (or filter) beside ordinary ones.  The
    outputs that see nothing else have float32's error."""
    import torch
    g = torch.Generator().manual_seed(Cin + 2)
    X, F = torch.randn((N, Cin, H, W), generator=g), torch.randn((Cout, Cin, k, k), generator=g)
    (X[N // 2] if which == "input" else F[Cout // 2]).mul_(size)
    want = dense64(X, F, stride)
    got = dense_gpu(X, F, stride, want)
    if which == "input":
        small, rest = (got[N // 2], want[N // 2]), (got[:N // 2], want[:N // 2])
    else:
        small, rest = (got[:, Cout // 2], want[:, Cout // 2]), (got[:, :Cout // 2], want[:, :Cout // 2])
    for y, ref in (small, rest):
        assert float((y - ref).norm(dtype=torch.float64) / ref.norm()) <= 1e-6   # as whole layers: up to 3600 terms


@pytest.mark.parametrize("k,stride,Cin,Cout,H,W,N", [SPLIT[0], SPLIT[4], SPLIT[5]])
@pytest.mark.parametrize("large", [1e20, 1e33, -3e38])
def test_small_operands_beside_large_ones(k, stride, Cin, Cout, H, W, N, large):
    """A tile with a number of 1e-36 is worked out on larger operands, where a large one, or a sum with it, may overflow: the
    outputs that see both, or either, are float32's, and all others are what they were without either."""
    import torch
    g = torch.Generator().manual_seed(Cin + 4)
    X, F = torch.randn((N, Cin, H, W), generator=g), torch.rand((Cout, Cin, k, k), generator=g) * 0.5 + 0.25
    plain = dense_gpu(X, F, stride, dense64(X[:1], F, stride).expand(N, -1, -1, -1))
    X[1, 0, 2, 4], X[1, Cin - 1, 2, 4], X[1, 1, 4, 2] = 1.1e-36, large, -1.3e-36
    want = dense64(X, F, stride)
    got = dense_gpu(X, F, stride, want)
    sees = (want - dense64(torch.where(X.abs() > 1e10, 0.0, X), F, stride)) != 0
    assert bool(sees.any()) and bool((~sees[1]).any())
    assert float(((got - want)[sees] / want[sees]).abs().max()) <= 1e-6
    assert float((got - want)[~sees].norm() / want[~sees].norm()) <= 1e-6
    assert torch.equal(got[2:], plain[2:])


@pytest.mark.parametrize("k,stride,Cin,Cout,H,W,N", [SPLIT[1], SPLIT[5]])
@pytest.mark.parametrize("bits", [0x7f800001, 0x7fc00000, 0xff80ffff - 2 ** 32, 0x7f800000])
def test_numbers_that_are_none(k, stride, Cin, Cout, H, W, N, bits):
    """A NaN, whichever bits it has set, reaches the outputs that see it as one, an infinity as an infinity or (times zero)
    a NaN, and all others are what they were."""
    import torch
    g = torch.Generator().manual_seed(Cin + 3)
    X, F = torch.randn((N, Cin, H, W), generator=g), torch.rand((Cout, Cin, k, k), generator=g) + 0.5
    F[3] = 0
    want = dense64(X, F, stride)
    plain = dense_gpu(X, F, stride, want)
    X.view(torch.int32)[2, Cin - 1, 5, 6] = bits
    got = dense_gpu(X, F, stride, want)
    sees = torch.zeros(want.shape, dtype=torch.bool)
    sees[2, :, 5 - k // 2:6 + k // 2, 6 - k // 2:7 + k // 2] = True
    assert torch.equal(got[~sees], plain[~sees])
    one = got[sees].reshape(Cout, -1)
    assert bool(torch.isnan(one[3]).all())
    one = one[torch.arange(Cout) != 3]
    assert bool(((one == float("inf")) if bits == 0x7f800000 else torch.isnan(one)).all())


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
