"""Launches that would leave compute units idle, in the kernels that walk chunks of channels (3x3, and 1x1 of many input
channels): wavefronts share a group's columns, the partial sums meet in LDS.  Group counts around the number of
wavefronts, ragged groups and chunks, chunks wider than a thread's loads ahead, every group size, residual and
activation, against the oracle."""
import numpy as np
import pytest

import oracle
import paper_2109_00170_amd as alcs
import workloads
from gpu_util import assert_close_after_activation

pytestmark = pytest.mark.gpu


def check(L, seed, bundle_waves=None, options=None):
    import torch
    d = workloads.make_layer(L, seed, with_bias=True)
    packed = alcs.alcs_pack_weights(d.W, d.mask, L.V, options=options)
    X, b = torch.from_numpy(d.X).cuda(), torch.from_numpy(d.bias).cuda()
    R = np.random.default_rng(seed).standard_normal((L.N, L.Cout, L.Ho, L.Wo)).astype(np.float32)
    for residual, act in ((None, None), (R, "relu6")):
        Y = torch.full((L.N, L.Cout, L.Ho, L.Wo), float("nan"), device="cuda")
        if residual is None:
            alcs.alcs_sparse_conv(packed, X, b, Y, stride=L.stride)
        else:
            Y.copy_(torch.from_numpy(R))
            alcs.alcs_sparse_conv_fused(packed, X, b, Y, Y, stride=L.stride, activation=act)  # the residual may be Y itself
        torch.cuda.synchronize()
        info = alcs.alcs_last_launch()
        if bundle_waves is not None:
            assert info["bundle_waves"] == bundle_waves, info
        got = Y.cpu().numpy()
        assert not np.isnan(got).any(), (L, info)
        ref = oracle.sparse_conv(d.W, d.mask, d.X, L.V, bias=d.bias, stride=L.stride, residual=residual, act=act)
        pre = oracle.sparse_conv(d.W, d.mask, d.X, L.V, bias=d.bias, stride=L.stride, residual=residual)
        assert_close_after_activation(got, ref, pre, "%s %s" % (L, info))
    packed.free()


# one image of 7x7 is one tile (stride 2: of 13x13): up to 256 groups make one round of one group each
@pytest.mark.parametrize("V", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("stride,Cin,shared", [(1, 70, True), (1, 70, False), (2, 70, True), (2, 530, False)])
def test_3x3_one_tile(V, stride, Cin, shared):
    L = workloads.Layer("few", Cin, 40 * V - (V > 1), 7 if stride == 1 else 13, 7 if stride == 1 else 12, k=3, stride=stride, N=1,
                        V=V, sparsity=0.7, w_std=0.1, tap_shared=shared)
    check(L, 8100 + V + Cin + stride, bundle_waves=16)


@pytest.mark.parametrize("groups,N,waves", [(64, 1, 16), (64, 5, 8), (64, 11, 4), (64, 20, 2), (63, 33, 1), (40, 60, 1)])
def test_3x3_wavefronts_per_group(groups, N, waves):
    L = workloads.Layer("share", 36, 4 * groups - 1, 8, 8, k=3, N=N, V=4, sparsity=0.8, w_std=0.1)
    check(L, 8200 + groups + N, bundle_waves=waves)


@pytest.mark.parametrize("H,W,shared", [(14, 14, True), (30, 17, False), (12, 40, True)])
def test_3x3_two_pixels_per_lane(H, W, shared):
    check(workloads.Layer("tall", 33, 30, H, W, k=3, N=1, V=4, sparsity=0.6, w_std=0.1, tap_shared=shared), 8300 + H + W)


def test_3x3_chunks_wider_than_the_loads_ahead():
    L = workloads.Layer("wide", 150, 20, 9, 9, k=3, stride=2, N=1, V=4, sparsity=0.7, w_std=0.1)
    check(L, 8400, options={"chunk_channels": 70})


@pytest.mark.parametrize("V", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("N,Cin", [(1, 2700), (17, 2561), (33, 2815), (70, 2600)])
def test_fully_connected_chunks(V, N, Cin):
    check(workloads.Layer("fc", Cin, 12 * V + 1, 1, 1, N=N, V=V, sparsity=0.9, w_std=0.05), 8500 + V + N)


@pytest.mark.parametrize("V,H,W,stride", [(2, 6, 6, 1), (2, 5, 5, 1), (1, 9, 7, 2), (2, 1, 3, 1)])
def test_1x1_chunks_on_images(V, H, W, stride):
    check(workloads.Layer("pw", 700, 30, H, W, stride=stride, N=2, V=V, sparsity=0.8, w_std=0.1), 8600 + H + W)


# launches of more workgroups than compute units whose chunks leave room for one workgroup on each
@pytest.mark.parametrize("V,groups,stride,H,shared,waves", [(4, 5, 1, 12, False, 2), (4, 17, 1, 12, True, 1), (8, 16, 1, 12, False, 1),
                                                            (1, 33, 2, 13, False, 1), (16, 3, 2, 13, True, 4), (2, 1, 2, 13, True, 16)])
def test_3x3_large_chunks_in_many_workgroups(V, groups, stride, H, shared, waves):
    L = workloads.Layer("alone", 75, V * groups - (V > 1), H, H, k=3, stride=stride, N=259, V=V, sparsity=0.8, w_std=0.1, tap_shared=shared)
    check(L, 8700 + V + groups, bundle_waves=waves, options={"chunk_channels": 64})
