"""How the 1x1 kernels reach their pixels (csrc/alcs_sparse.hip, Access): quads at any address with a
seam between two images, images of one pixel (fully connected layers) transposed on the way into
LDS, and the kernels whose wavefronts share bundles - at the sizes where each can go wrong, with a
residual and an activation, in float32 and on bfloat16 tensors, against the oracle."""
import pytest

import workloads
from test_gpu_bf16 import run_bf16
from test_gpu_fused_epilogue import run_fused

pytestmark = pytest.mark.gpu

# every remainder of the pixel count by 4, the smallest image of a quad, quads over the seam of two
# images and at the end of the last one
SEAMS = [(2, 2, 5), (1, 5, 7), (1, 5, 1), (2, 3, 9), (7, 7, 3), (7, 1, 6), (9, 5, 2), (3, 13, 11), (45, 37, 1)]


@pytest.mark.parametrize("H,W,N", SEAMS)
@pytest.mark.parametrize("V,pv", [(1, 2), (2, 4), (4, 1), (4, 2), (4, 4), (8, 2), (16, 1)])
def test_unaligned_quads(H, W, N, V, pv):
    L = workloads.Layer("seam", 37, 21, H, W, N=N, V=V, sparsity=0.5, w_std=0.3)
    run_fused(L, 6000 + 10 * H + W + V, "relu", pv=pv)
    run_bf16(L, 6000 + 10 * H + W + V, act="relu6", with_res=True, pv=pv)


@pytest.mark.parametrize("Cin,V,slots", [(520, 4, 4), (700, 8, 2), (1300, 16, 4)])
@pytest.mark.parametrize("H,W,N", [(7, 7, 3), (1, 5, 9), (13, 3, 2)])
def test_unaligned_quads_several_groups_per_wavefront(Cin, V, slots, H, W, N):
    L = workloads.Layer("seam_gs", Cin, 70, H, W, N=N, V=V, sparsity=0.9, w_std=0.1)
    run_fused(L, 6100 + Cin + H, None, pack_tuning={"group_slots": slots})
    run_bf16(L, 6100 + Cin + H, act=None, with_res=True, pack_tuning={"group_slots": slots})


@pytest.mark.parametrize("Cin,Cout,V", [(16, 10, 4), (63, 33, 8), (130, 40, 1), (511, 24, 4), (513, 30, 4), (1025, 100, 8),
                                        (2558, 20, 16), (700, 12, 2), (2600, 17, 4)])
@pytest.mark.parametrize("N", [1, 15, 17, 40, 130])
def test_rows(Cin, Cout, V, N):
    """Fully connected: channels that are no multiple of 4 or 16, rows that are no multiple of 16 and of one to
    four groups of 16, ragged groups, the kernels that stream their channels in chunks."""
    L = workloads.Layer("rows", Cin, Cout, 1, 1, N=N, V=V, sparsity=0.8, w_std=0.1)
    run_fused(L, 6200 + Cin + N, "relu")
    if Cin <= (2558 if V >= 4 else 639):
        run_bf16(L, 6200 + Cin + N, act="relu", with_res=True)


@pytest.mark.parametrize("Cin,Cout,V,H,N,stride", [(512, 512, 4, 14, 1, 1), (512, 96, 8, 7, 1, 1), (1024, 1024, 4, 7, 1, 1),
                                                   (512, 64, 16, 14, 2, 2), (640, 40, 4, 5, 1, 1), (1300, 260, 8, 4, 2, 1)])
@pytest.mark.parametrize("waves", [0, 4])
def test_wavefronts_share_bundles(Cin, Cout, V, H, N, stride, waves):
    """Few pixel tiles: fewer bundles per workgroup than wavefronts; segments shorter than the share of
    a wavefront leave some of them without columns."""
    for sparsity in (0.7, 0.99):
        L = workloads.Layer("share", Cin, Cout, H, H, N=N, V=V, stride=stride, sparsity=sparsity, w_std=0.1)
        info = run_fused(L, 6300 + Cin + H, "relu6", waves=waves)
        # (at 99 % the longest segments may be one run of 16 columns, which nobody shares)
        assert sparsity > 0.9 or info["bundle_waves"] > 1, info
