"""Launches that fill the chip, with group counts that are no multiple of what the workgroups hold: the groups are dealt
evenly to the group tiles and to their wavefronts (3x3, and 1x1 kernels that walk chunks of channels)."""
import numpy as np
import pytest

import workloads
from gpu_util import TOL, assert_close_after_activation, oracle_ref, rel_err, run_sparse

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,groups", [(1, 33), (2, 17), (4, 1), (4, 9), (4, 17), (4, 33), (4, 65), (8, 17), (16, 33)])
@pytest.mark.parametrize("shared", [False, True])
def test_3x3(V, groups, shared):
    L = workloads.Layer("deal3", 9, V * groups - (V > 1), 8, 8, k=3, N=257, V=V, sparsity=0.7, w_std=0.2, tap_shared=shared)
    d = workloads.make_layer(L, 9600 + V + groups, with_bias=True)
    got, info = run_sparse(d)
    assert info["bundle_waves"] == 1 and rel_err(got, oracle_ref(d)) <= TOL, info


@pytest.mark.parametrize("V,groups", [(1, 33), (2, 9), (2, 17), (2, 40), (2, 65)])
def test_1x1_chunks(V, groups):
    L = workloads.Layer("deal1", 660, V * groups - (V > 1), 8, 8, N=257, V=V, sparsity=0.9, w_std=0.1)
    d = workloads.make_layer(L, 9700 + V + groups, with_bias=True)
    got, info = run_sparse(d)
    assert info["mode"] == 2 and rel_err(got, oracle_ref(d)) <= TOL, info


# The kernel whose wavefronts own several groups (launches of few workgroups take another by themselves: groups_per_wave asks for
# this one), every group size and way of reading the images: aligned, unaligned, one pixel at a time, one-pixel images.
@pytest.mark.parametrize("V,Cin,chunk", [(1, 650, 0), (2, 700, 0), (4, 100, 33), (8, 130, 64), (16, 70, 33)])
@pytest.mark.parametrize("H,W,stride,N", [(12, 12, 1, 3), (7, 7, 1, 5), (9, 7, 2, 4), (1, 1, 1, 70)])
@pytest.mark.parametrize("ug", [2, 4])
def test_1x1_chunks_several_groups_per_wavefront(V, Cin, chunk, H, W, stride, N, ug):
    import oracle
    import paper_2109_00170_amd as alcs
    import torch
    L = workloads.Layer("own", Cin, 35 * V - (V > 1), H, W, stride=stride, N=N, V=V, sparsity=0.8, w_std=0.1)
    d = workloads.make_layer(L, 9800 + V + H + ug, with_bias=True)
    options = {"groups_per_wave": ug, "chunk_channels": chunk}
    got, info = run_sparse(d, options=options)
    assert (info["mode"], info["bundle_waves"], info["waves"], info["pv"]) == (2, 1, 8, 1) and info["group_tiles"] == (3 if ug == 2 else 2), info
    assert rel_err(got, oracle_ref(d)) <= TOL
    R = np.random.default_rng(V).standard_normal((N, L.Cout, L.Ho, L.Wo)).astype(np.float32)
    packed = alcs.alcs_pack_weights(d.W, d.mask, V, options=options)
    Y = torch.full(R.shape, float("nan"), device="cuda")
    alcs.alcs_sparse_conv_fused(packed, torch.from_numpy(d.X).cuda(), torch.from_numpy(d.bias).cuda(), torch.from_numpy(R).cuda(), Y,
                                stride=stride, activation="relu")
    torch.cuda.synchronize()
    assert alcs.alcs_last_launch()["mode"] == 2 and alcs.alcs_last_launch()["bundle_waves"] == 1
    ref = oracle.sparse_conv(d.W, d.mask, d.X, V, bias=d.bias, stride=stride, residual=R, act="relu")
    pre = oracle.sparse_conv(d.W, d.mask, d.X, V, bias=d.bias, stride=stride, residual=R)
    assert_close_after_activation(Y.cpu().numpy(), ref, pre, str(info))
    packed.free()
