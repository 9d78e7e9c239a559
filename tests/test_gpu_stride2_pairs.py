"""1x1 layers at stride 2 over images whose width is a multiple of 4 and whose output has a multiple of 4 pixels: pairs of
neighbours are read 16 bytes (bfloat16: 8) at a time.  Rows of two, four and fourteen output pixels (quads that end with a
row, or wrap into the next one), odd heights, channel counts around a thread's loads in flight, several groups per wavefront,
and the last row and image, whose reads end with the tensor."""
import pytest

import workloads
from gpu_util import TOL, oracle_ref, rel_err, run_sparse
from test_gpu_bf16 import run_bf16
from test_gpu_math16 import run_m16

pytestmark = pytest.mark.gpu

IMAGES = [(4, 4), (7, 4), (3, 8), (28, 28), (27, 28), (5, 56)]


def layer(Cin, H, W, N, V, Cout=27):
    return workloads.Layer("s2_%d_%dx%d" % (Cin, H, W), Cin, Cout, H, W, stride=2, N=N, V=V, sparsity=0.7, w_std=0.2)


@pytest.mark.parametrize("H,W", IMAGES + [(10, 12), (6, 6), (9, 9)])  # (the last three are read one pixel at a time)
@pytest.mark.parametrize("V,Cin", [(1, 37), (2, 5), (4, 64), (8, 33), (16, 129), (4, 530), (8, 1300)])
def test_float32(V, Cin, H, W):
    d = workloads.make_layer(layer(Cin, H, W, 3, V), 9100 + V + H + W, with_bias=True)
    got, info = run_sparse(d)
    assert info["mode"] == 1
    assert rel_err(got, oracle_ref(d)) <= TOL, info


@pytest.mark.parametrize("pv", [1, 2, 4])
def test_pixels_per_lane(pv):
    d = workloads.make_layer(layer(40, 28, 28, 5, 4), 9200 + pv, with_bias=True)
    got, info = run_sparse(d, options={"pv": pv})
    assert info["pv"] == pv and rel_err(got, oracle_ref(d)) <= TOL, info


@pytest.mark.parametrize("H,W", IMAGES)
@pytest.mark.parametrize("Cin", [33, 540])
def test_bfloat16_tensors(Cin, H, W):
    run_bf16(layer(Cin, H, W, 6, 4), 9300 + Cin + H + W, act="relu", with_res=True)


@pytest.mark.parametrize("H,W", IMAGES)
@pytest.mark.parametrize("V,Cin", [(4, 33), (8, 640), (16, 97)])
def test_16bit_arithmetic(V, Cin, H, W):
    run_m16(layer(Cin, H, W, 6, V), 9400 + Cin + H + W, act="relu6", with_res=True)
    run_m16(layer(Cin, H, W, 6, V), 9500 + Cin + H + W, options={"pv": 1})


def check_forms(L, seed, options, want):
    """The plain and the fused call (residual and activation) against the oracle; `want`: what the launch has to report."""
    import numpy as np
    import oracle
    import paper_2109_00170_amd as alcs
    import torch
    from gpu_util import assert_close_after_activation
    d = workloads.make_layer(L, seed, with_bias=True)
    packed = alcs.alcs_pack_weights(d.W, d.mask, L.V, options=options)
    X, b = torch.from_numpy(d.X).cuda(), torch.from_numpy(d.bias).cuda()
    R = np.random.default_rng(seed).standard_normal((L.N, L.Cout, L.Ho, L.Wo)).astype(np.float32)
    for residual, act in ((None, None), (R, "relu6")):
        Y = torch.full((L.N, L.Cout, L.Ho, L.Wo), float("nan"), device="cuda")
        if residual is None:
            alcs.alcs_sparse_conv(packed, X, b, Y, stride=2)
        else:
            alcs.alcs_sparse_conv_fused(packed, X, b, torch.from_numpy(R).cuda(), Y, stride=2, activation=act)
        torch.cuda.synchronize()
        info = alcs.alcs_last_launch()
        assert {k: info[k] for k in want} == want, info
        ref = oracle.sparse_conv(d.W, d.mask, d.X, L.V, bias=d.bias, stride=2, residual=residual, act=act)
        pre = oracle.sparse_conv(d.W, d.mask, d.X, L.V, bias=d.bias, stride=2, residual=residual)
        got = Y.cpu().numpy()
        assert not np.isnan(got).any()
        assert_close_after_activation(got, ref, pre, "%s %s" % (L, info))
    packed.free()
    return info


# channels in chunks, the last one ragged: a launch of a few workgroups (wavefronts share groups) and one that fills the chip
@pytest.mark.parametrize("V,Cin,chunk", [(1, 700, 0), (2, 650, 0), (4, 130, 50), (8, 101, 100), (16, 70, 33)])
@pytest.mark.parametrize("H,W,N", [(4, 4, 3), (27, 28, 2), (28, 28, 95)])
def test_chunks(V, Cin, chunk, H, W, N):
    L = layer(Cin, H, W, N, V, Cout=5 * V + (V > 1))
    check_forms(L, 9600 + V + Cin + H, {"chunk_channels": chunk} if chunk else None, {"mode": 2})
    if N == 95:  # the kernel whose wavefronts own groups
        check_forms(L, 9600 + V + Cin + H, {"chunk_channels": chunk, "groups_per_wave": 2}, {"mode": 2, "bundle_waves": 1})


@pytest.mark.parametrize("slots,pv,N", [(4, 2, 95), (4, 1, 95), (2, 2, 20), (2, 1, 20), (4, 2, 3)])
def test_several_groups_per_wavefront(slots, pv, N):
    # (95 images of 14x14 outputs in tiles of 32 pixels: more than two rounds of workgroups, planes that end off the cache lines)
    info = check_forms(layer(40, 28, 28, N, 4, Cout=37), 9700 + slots + pv, {"group_slots": slots, "pv": pv}, {"mode": 1, "group_slots": slots, "pv": pv})
    assert N < 95 or info["workgroups"] > 512
