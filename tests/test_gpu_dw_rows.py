"""Depthwise 3x3 with four pixels of a row per lane (csrc/alcs_dw_strip.h) at the sizes where it can go
wrong, in the stand-alone layer and as the stage of the fused block: widths that are no multiple of what
the lanes read, rows of several images in a tile or a wavefront, fewer channels or planes than a wavefront
takes, several passes over a tile, rows wider than a wavefront; and wavefronts that share bundles."""
import numpy as np
import pytest

import oracle
import paper_2109_00170_amd as alcs
import workloads
from gpu_util import TOL, rel_err
from test_gpu_dw_block import dw_inputs, run_block

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stride", [1, 2])
@pytest.mark.parametrize("C,N,H,W", [(3, 2, 3, w) for w in range(4, 18)] + [
    (70, 1, 7, 7), (5, 5, 7, 7), (1, 1, 1, 5), (9, 1, 64, 4), (3, 1, 65, 4), (2, 3, 30, 31),
    (2, 1, 5, 255), (2, 1, 4, 257), (3, 1, 3, 500), (2, 1, 3, 513), (1, 2, 2, 1031),
    (13, 40, 60, 131), (11, 16, 90, 260), (20, 41, 22, 27)])   # large, with half of the lanes idle as rows or nearly none
def test_layer(C, N, H, W, stride):
    import torch
    D, X, b = dw_inputs(C, N, H, W, 31 * C + W)
    Ho, Wo = oracle.out_size(H, 3, stride), oracle.out_size(W, 3, stride)
    Y = torch.full((N, C, Ho, Wo), float("nan"), dtype=torch.float32, device="cuda")
    alcs.alcs_depthwise_conv(torch.from_numpy(D).cuda(), torch.from_numpy(X).cuda(), torch.from_numpy(b).cuda(), Y,
                             stride=stride)
    got = Y.cpu().numpy()
    assert not np.isnan(got).any()
    assert rel_err(got, oracle.depthwise(D, X, bias=b, stride=stride)) <= TOL


@pytest.mark.parametrize("stride", [1, 2])
@pytest.mark.parametrize("Cin,H,W,N,pv", [
    (33, 5, 5, 40, 4),      # 51 rows a tile: four passes of a wavefront
    (1, 9, 8, 3, 1),        # one channel, eight channels' lanes
    (7, 14, 14, 5, 2), (29, 7, 7, 9, 4), (18, 3, 13, 7, 1), (40, 12, 15, 4, 2), (21, 6, 50, 3, 1), (5, 3, 63, 3, 1),
    (9, 14, 14, 80, 1),     # whole rows would make a second round of the chip
    (4, 56, 56, 10, 0),     # few input channels: pixel pairs at stride 2 too
    (12, 4, 100, 2, 2), (9, 2, 121, 2, 4), (10, 3, 250, 2, 4), (16, 28, 28, 2, 4), (130, 2, 4, 3, 4),
    # rows of several images: one-row images, an odd first row, the last image's odd row (in pairs: see below)
    (6, 1, 16, 9, 1), (13, 4, 21, 5, 1), (14, 5, 10, 7, 2), (17, 3, 4, 11, 4),
    (19, 6, 17, 3, 1), (23, 4, 30, 4, 2)])   # widths of every remainder
def test_block_on_whole_rows(Cin, H, W, N, pv, stride):
    Hin, Win = (H, W) if stride == 1 else (2 * H - H % 2, 2 * W - W % 2)   # odd and even inputs
    L = workloads.Layer("rows", Cin, 20, H, W, N=N, V=4, sparsity=0.5, w_std=0.3)
    run_block(L, Hin, Win, stride, 7000 + Cin + W, pv=pv)


def in_pairs(Cin, H, W, N, pv, waves):
    """Whether the stage works out two rows per lane (stride 1): the launcher's rule."""
    rows = min(64 * pv // W, N * H)
    while rows < N * H and H * W % 4 == 0 and rows * W % 4:
        rows -= 1
    assert 4 * rows * W >= 3 * 64 * pv or rows == N * H, "tiles are not whole rows"
    quads = -(-W // 4)

    def turns(k):
        sets = -(-rows // k)
        lanes = min(sets, 64 // quads) * quads
        return -(-(-(-Cin // min(64 // lanes, Cin))) // waves) * -(-sets // (64 // quads))
    return rows > 1 and 8 * turns(2) <= 5 * turns(1)


@pytest.mark.parametrize("Cin,H,W,N,pv", [
    (64, 1, 16, 9, 1), (90, 1, 5, 40, 2), (61, 1, 9, 29, 4),      # one-row images: every pair lies in two of them
    (64, 3, 16, 7, 1), (40, 5, 10, 7, 2), (33, 7, 7, 9, 4), (66, 3, 4, 21, 1),   # pairs over a seam, on odd and even rows
    (70, 3, 21, 5, 1), (50, 6, 30, 3, 2),                           # an odd number of rows in a tile
    (17, 3, 11, 1, 2), (48, 9, 14, 1, 2)])                          # the only image's odd row
def test_pairs_of_rows(Cin, H, W, N, pv):
    L = workloads.Layer("pairs", Cin, 20, H, W, N=N, V=4, sparsity=0.5, w_std=0.3)
    info = run_block(L, H, W, 1, 7100 + Cin + W, pv=pv, waves=2)
    assert in_pairs(Cin, H, W, N, info["pv"], info["waves"]), info


@pytest.mark.parametrize("Cin,Cout,hw,N,V,sparsity,one", [
    (23, 74, 28, 17, 4, 0.9, True),       # four group tiles, four pixels per lane, few channels
    (104, 24, 14, 84, 2, 0.6, False),     # three, 104 channels: the two layers
    (122, 22, 56, 7, 2, 0.5, True),       # two
    (153, 60, 7, 34, 4, 0.8, True)])      # three or four, one pixel per lane
def test_group_tiles_that_work_the_stage_out_again(Cin, Cout, hw, N, V, sparsity, one):
    L = workloads.Layer("again", Cin, Cout, hw, hw, N=N, V=V, sparsity=sparsity, w_std=0.2)
    info = run_block(L, hw, hw, 1, 7200 + Cin, act="relu", workspace=True, expect_mode=1 if one else None)
    if one:
        assert info["group_tiles"] > 1, info


@pytest.mark.parametrize("Cin,slots,hw,stride,N", [(520, 4, 14, 1, 2), (600, 2, 7, 2, 3), (1100, 4, 7, 1, 40), (520, 4, 3, 1, 5)])
def test_block_wavefronts_share_bundles(Cin, slots, hw, stride, N):
    L = workloads.Layer("split", Cin, 90, hw, hw, N=N, V=4, sparsity=0.9, w_std=0.1)
    info = run_block(L, hw * stride, hw * stride, stride, 7300 + Cin, pack_tuning={"group_slots": slots}, with_res=True,
                     act="relu")
    assert info["bundle_waves"] > 1, info
