"""The dense convolution's small launches (k_dense_few: 32 x 32 outputs a workgroup, sixteen wavefronts that share the
channels), and the tiles of float32 in launches too large for it."""
import numpy as np
import pytest

import workloads
from gpu_util import TOL, oracle_ref, rel_err, run_dense

pytestmark = pytest.mark.gpu


def check(k, stride, Cin, Cout, H, W, N, bias=True):
    L = workloads.Layer("few", Cin, Cout, H, W, k=k, stride=stride, N=N, V=1, sparsity=0.0, w_std=0.1, mask_kind="none")
    d = workloads.make_layer(L, 8900 + Cin + Cout + H, with_bias=bias)
    got = run_dense(d)
    assert not np.isnan(got).any()
    assert rel_err(got, oracle_ref(d)) <= TOL


# channels around the wavefronts' units (two channels of 3x3, eight of 1x1, sixteen wavefronts), rows and pixels around the
# tile, images smaller than it, both strides, the largest launch (256 tiles)
@pytest.mark.parametrize("Cin", [1, 2, 3, 31, 32, 33, 65, 130])
@pytest.mark.parametrize("stride,Cout,H,W,N", [(1, 1, 1, 1, 1), (1, 31, 4, 8, 1), (2, 33, 7, 5, 3), (1, 32, 11, 3, 2), (2, 64, 2, 2, 17)])
def test_3x3(Cin, stride, Cout, H, W, N):
    check(3, stride, Cin, Cout, H, W, N, bias=Cin != 3)


@pytest.mark.parametrize("Cin", [1, 7, 8, 9, 127, 128, 129, 300])
@pytest.mark.parametrize("stride,Cout,H,W,N", [(1, 1, 1, 1, 1), (1, 31, 4, 8, 1), (2, 33, 7, 5, 3), (1, 32, 11, 3, 2), (2, 64, 2, 2, 17)])
def test_1x1(Cin, stride, Cout, H, W, N):
    check(1, stride, Cin, Cout, H, W, N, bias=Cin != 7)


# (a launch of one round of small tiles, and the next larger one, which is not left to k_dense_few)
ONE_ROUND = [((k, 1, 20, 32, 4, 8, N), kind) for k in (1, 3) for N, kind in ((256, "few"), (257, "float32"))]


@pytest.mark.parametrize("k", [1, 3])
@pytest.mark.parametrize("N", [256, 257])
def test_around_one_round(k, N):
    check(k, 1, 20, 32, 4, 8, N)


# one shape for each float32 tile (and the gather) that test_dense_tiles names, in launches of more than one round of small tiles
LARGER = [
    (3, 1, 8, 32, 12, 11, 63), (3, 1, 9, 31, 4, 4, 513), (3, 1, 24, 33, 1, 1, 4097), (3, 1, 16, 65, 3, 2, 454), (3, 2, 17, 130, 15, 9, 41),
    (3, 2, 12, 40, 33, 58, 9), (3, 1, 5, 20, 3, 300, 10), (3, 2, 3, 32, 40, 224, 4), (3, 2, 8, 64, 64, 203, 2), (3, 2, 13, 300, 31, 146, 1),
    (1, 1, 16, 16, 5, 3, 547), (1, 1, 32, 16, 5, 3, 547), (1, 1, 8, 40, 6, 5, 137), (1, 1, 31, 64, 1, 1, 4097), (1, 2, 64, 30, 31, 17, 57)]


@pytest.mark.parametrize("k,stride,Cin,Cout,H,W,N", LARGER)
def test_tiles_of_larger_launches(k, stride, Cin, Cout, H, W, N):
    check(k, stride, Cin, Cout, H, W, N)
