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
