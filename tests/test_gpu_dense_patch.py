"""The dense convolution's tiles (csrc/alcs_dense.hip) at the sizes where they can go wrong, against the
oracle: channels that are no multiple of a step, channel and pixel tiles with a remainder, tiles over
several images, every number of staged positions per thread, and the images that fall to the
word-by-word kernel."""
import numpy as np
import pytest

import workloads
from gpu_util import TOL, oracle_ref, rel_err, run_dense

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,stride,Cin,Cout,H,W,N", [
    (3, 1, 8, 32, 12, 11, 1),      # one step of 8 channels
    (3, 1, 9, 31, 4, 4, 40),       # a step and a channel; 8 images in a tile
    (3, 1, 24, 33, 1, 1, 300),     # one-pixel images: 128 a tile, past the staging
    (3, 1, 16, 65, 3, 2, 25),      # 21 images in a tile
    (3, 2, 17, 130, 15, 9, 5),
    (3, 2, 12, 40, 33, 58, 3),     # more than 512 staged positions
    (3, 1, 10, 70, 13, 140, 2),    # 768 to 1024 of them
    (3, 1, 5, 20, 3, 300, 2),      # wider than the staging
    (3, 2, 3, 32, 40, 224, 2),
    (1, 1, 32, 16, 5, 3, 9),       # one step of 32 channels
    (1, 1, 31, 64, 1, 1, 70),
    (1, 1, 97, 129, 9, 7, 31),
    (1, 2, 64, 30, 31, 17, 6),
    (1, 1, 160, 200, 56, 56, 5),   # several tiles a compute unit
    (3, 1, 64, 256, 30, 30, 12),   # 128 x 128
])
def test_dense_tiles(k, stride, Cin, Cout, H, W, N):
    L = workloads.Layer("tile", Cin, Cout, H, W, k=k, stride=stride, N=N, V=1, sparsity=0.0, w_std=0.1,
                        mask_kind="none")
    d = workloads.make_layer(L, 8800 + Cin + Cout, with_bias=True)
    got = run_dense(d)
    assert not np.isnan(got).any()
    assert rel_err(got, oracle_ref(d)) <= TOL
