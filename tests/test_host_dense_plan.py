"""The dense convolution's choice of kernel and tile (csrc/alcs_dense_plan.h): every tile it can choose is run by the GPU
tests, and what it says of a tile is what the kernel takes."""
import math
import random

from dense_plan import dense_plan
from test_gpu_dense_few import LARGER, ONE_ROUND
from test_gpu_dense_patch import SPLIT, TILES

# (kernel, kind, channels, pixels, staged positions per thread) of the kernels alcs_dense.hip has
KERNELS = ({(1, "split", 128, bn, 1) for bn in (256, 128)} | {(1, "float32", 64, 64, 1), (1, "float32", 32, 128, 1)} |
           {(3, "split", 128, 256, 1)} | {(3, "split", bm, 128, n) for bm in (128, 64) for n in (1, 2)} |
           {(3, "float32", 128, 128, 3), (3, "float32", 128, 128, 4), (3, "float32", 64, 128, 2)} |
           {(3, "float32", 32, 128, n) for n in (2, 3, 4)} | {(3, "float32", 64, 64, n) for n in (3, 4)} |
           {(3, "gather", 64, 128, 0), (3, "gather", 128, 128, 0)} | {(k, "few", 32, 32, 0) for k in (1, 3)})


def shapes(n):
    rng = random.Random(7)

    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    for _ in range(n):
        yield (rng.choice([1, 3, 3, 3]), rng.choice([1, 2]), log(3, 1024), log(8, 1024), log(1, 230), log(1, 260), log(1, 300))


def test_every_tile_that_can_be_chosen_is_tested():
    tested = {dense_plan(*t)[0] for t in TILES + LARGER}
    chosen = {dense_plan(*t)[0] for t in shapes(100000)}
    assert chosen <= tested, chosen - tested
    assert tested == KERNELS, tested ^ KERNELS
    assert all(dense_plan(*t)[0][1] != "few" for t in LARGER)
    assert {dense_plan(*t)[0] for t in SPLIT} == {p for p in KERNELS if p[1] == "split"}


def test_a_tile_fits_what_its_kernel_stages():
    # (the last two: 900000 channels, too many bytes for a tile of 128 pixels and not for one of 64, whose kernel has room for
    # at least 513 positions)
    for t in list(shapes(20000)) + list(TILES) + [(3, 2, 900000, 64, 20, 20, 3), (3, 2, 900000, 9, 20, 20, 5)]:
        plan, npos, lds = dense_plan(*t, few=False)
        k, kind, bm, bn, npt = plan
        assert plan in KERNELS, (t, plan)
        if kind == "gather":
            continue
        assert lds <= 160 * 1024
        if k == 3:
            # input rows and images that a tile's pixels can touch, counted on every place where a tile may begin
            stride, H, W, N = t[1], t[4], t[5], t[6]
            Ho, Wo = (H + stride - 1) // stride, (W + stride - 1) // stride
            cols, worst = (Wo - 1) * stride + 3, 0
            for first in range(min(Ho * Wo, 400)):
                a, b = first // Wo, min(first + bn - 1, N * Ho * Wo - 1) // Wo
                rows = sum((min(b, (n + 1) * Ho - 1) - max(a, n * Ho)) * stride + 3 for n in range(a // Ho, b // Ho + 1))
                worst = max(worst, rows * cols)
            assert worst <= npos <= npt * (512 if kind == "split" else 256), (t, plan)


def test_small_launches_end_with_one_round():
    # 32 x 32 outputs to a workgroup, one workgroup to a compute unit
    for t, kind in ONE_ROUND:
        assert (dense_plan(*t)[0][1] == "few") == (kind == "few"), t
    for t in shapes(20000):
        k, stride, Cin, Cout, H, W, N = t
        tiles = -(-N * -(-H // stride) * -(-W // stride) // 32) * -(-Cout // 32)
        plan = dense_plan(*t, few=False)[0]
        assert (dense_plan(*t)[0][1] == "few") == (plan[1] != "split" and tiles <= 256), t
