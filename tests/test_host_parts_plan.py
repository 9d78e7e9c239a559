"""The kernels that walk chunks of channels: which launches give a wavefront one group, or a part of one
(csrc/alcs_parts_plan.h)."""
import math
import random

from parts_plan import groups_of_tile, parts_plan


def shapes(n):
    rng = random.Random(11)

    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    for _ in range(n):
        three = rng.random() < 0.6
        G, V = log(1, 1000), rng.choice([1, 2, 4, 8, 16])
        ug = 2 if G <= 16 or (three and V >= 8) else rng.choice([2, 4])
        strided = not three and rng.random() < 0.3
        yield dict(V=V, G=G, npt=log(1, 4000), ngt=-(-G // (8 * ug)), cols=log(1, 5000), nchunks=log(1, 20),
                   nw=16 if three or rng.random() < 0.3 else 8, three=three, alone=three and rng.random() < 0.3,
                   wide=three and V == 8 and rng.random() < 0.5, strided=strided,
                   stride2=strided or (not three and rng.random() < 0.3), uneven=rng.random() < 0.2)


def test_every_group_has_a_wavefront_and_every_wavefront_a_place():
    taken = 0
    for s in shapes(20000):
        p = parts_plan(**s)
        if p is None:
            continue
        taken += 1
        ngt, gpt, ks = p
        assert ngt * gpt >= s["G"] and (ngt - 1) * gpt < s["G"], (s, p)
        assert ks >= 1 and ks & (ks - 1) == 0 and gpt * ks <= s["nw"], (s, p)
        if s["npt"] * s["ngt"] >= 256:
            assert s["alone"], (s, p)
        else:
            assert ngt > s["ngt"], (s, p)
    assert taken > 4000


def test_small_groups_alone_on_their_compute_units():
    # more rounds of a multiply that is not short: as it was; a short one, few more rounds, or uneven groups: as parts
    big = dict(alone=True, nw=16)
    assert parts_plan(V=1, G=31, npt=448, ngt=1, cols=199 * 9, nchunks=9, **big) is None
    assert parts_plan(V=1, G=160, npt=182, ngt=5, cols=134 * 9, nchunks=9, **big) is None
    assert parts_plan(V=2, G=20, npt=448, ngt=1, cols=223 * 9, nchunks=9, **big) is None
    assert parts_plan(V=1, G=152, npt=168, ngt=5, cols=46 * 17, nchunks=17, **big) == (10, 16, 1)
    assert parts_plan(V=2, G=144, npt=54, ngt=5, cols=181 * 12, nchunks=12, **big) == (9, 16, 1)
    assert parts_plan(V=2, G=128, npt=168, ngt=4, cols=130 * 10, nchunks=10, uneven=True, **big) == (8, 16, 1)
    assert parts_plan(V=2, G=92, npt=136, ngt=3, cols=130 * 10, nchunks=10, uneven=True, **big) is None
    assert parts_plan(V=1, G=64, npt=324, ngt=2, cols=130 * 10, nchunks=10, uneven=True, **big) is None
    for V in (4, 8, 16):
        assert parts_plan(V=V, G=160, npt=182, ngt=5, cols=134 * 9, nchunks=9, **big) == (10, 16, 1)


def test_single_channels_with_a_shared_pattern():
    # longer turns of a wavefront's one group: fewer rounds are few more than for other patterns
    big = dict(V=1, alone=True, nw=16)
    for shared in (False, True):
        parts = dict(big, shared=shared)
        assert (parts_plan(G=648, npt=18, ngt=21, cols=267 * 12, nchunks=12, **parts) is None) == shared
        assert (parts_plan(G=440, npt=104, ngt=14, cols=60 * 14, nchunks=14, **parts) is None) == shared
        assert parts_plan(G=109, npt=212, ngt=4, cols=44 * 9, nchunks=9, **parts) == (7, 16, 1)
        assert parts_plan(G=110, npt=140, ngt=4, cols=79 * 17, nchunks=17, **parts) == (7, 16, 1)
    assert parts_plan(G=440, npt=104, ngt=14, cols=60 * 14, nchunks=14, alone=True, nw=16, V=2, shared=True) == (28, 16, 1)


def test_more_than_one_round():
    big = dict(alone=True, nw=16)
    assert parts_plan(V=4, G=22, npt=210, ngt=1, cols=76 * 17, nchunks=17, **big) is None
    assert parts_plan(V=4, G=43, npt=112, ngt=2, cols=46 * 10, nchunks=10, **big) is None
    assert parts_plan(V=1, G=118, npt=60, ngt=4, cols=202 * 11, nchunks=11, **big) is None
    assert parts_plan(V=4, G=80, npt=84, ngt=3, cols=178 * 13, nchunks=13, **big) == (5, 16, 1)
    assert parts_plan(V=4, G=56, npt=56, ngt=2, cols=244 * 11, nchunks=11, **big) == (4, 16, 1)
    assert parts_plan(V=2, G=268, npt=18, ngt=9, cols=167 * 11, nchunks=11, uneven=True, **big) == (17, 16, 1)
    assert parts_plan(V=1, G=268, npt=18, ngt=9, cols=167 * 11, nchunks=11, uneven=True, **big) is None
    assert parts_plan(V=4, G=138, npt=30, ngt=5, cols=120 * 13, nchunks=13, uneven=True, **big) == (9, 16, 1)
    assert parts_plan(V=4, G=17, npt=140, ngt=1, cols=120 * 13, nchunks=13, uneven=True, **big) is None
    rows = dict(three=False, nw=8)
    assert parts_plan(V=2, G=100, npt=50, ngt=4, cols=56, nchunks=4, strided=True, stride2=True, **rows) is None
    assert parts_plan(V=1, G=20, npt=181, ngt=1, cols=256, nchunks=4, stride2=True, **rows) is None
    assert parts_plan(V=2, G=80, npt=27, ngt=3, cols=570, nchunks=6, strided=True, stride2=True, **rows) == (10, 8, 1)
    assert parts_plan(V=1, G=32, npt=233, ngt=1, cols=452, nchunks=5, **rows) == (4, 8, 1)
    assert parts_plan(V=4, G=28, npt=245, ngt=1, cols=400, nchunks=16, **rows) is None
    assert parts_plan(V=1, G=136, npt=41, ngt=5, cols=147, nchunks=3, unaligned=True, **rows) is None
    assert parts_plan(V=2, G=136, npt=49, ngt=5, cols=284, nchunks=4, unaligned=True, **rows) == (17, 8, 1)
    assert parts_plan(V=4, G=52, npt=70, ngt=2, cols=640, nchunks=12, **rows) == (7, 8, 1)
    assert parts_plan(V=16, G=9, npt=136, ngt=1, cols=880, nchunks=14, **rows) is None
    assert parts_plan(V=2, G=16, npt=135, ngt=1, cols=234, nchunks=3, **rows) == (2, 8, 1)


def test_rows_staged_one_pixel_at_a_time():
    rows = dict(three=False, nw=8, strided=True, stride2=True)
    assert parts_plan(V=8, G=3, npt=19, ngt=1, cols=40 * 16, nchunks=16, **rows) is None
    assert parts_plan(V=2, G=11, npt=9, ngt=1, cols=42 * 5, nchunks=5, **rows) is None
    assert parts_plan(V=8, G=14, npt=11, ngt=1, cols=26 * 15, nchunks=15, **rows) is None
    assert parts_plan(V=8, G=3, npt=1, ngt=1, cols=40 * 16, nchunks=16, **rows) == (3, 1, 8)
    assert parts_plan(V=2, G=15, npt=6, ngt=1, cols=72 * 5, nchunks=5, **rows) == (15, 1, 8)
    assert parts_plan(V=8, G=27, npt=7, ngt=1, cols=13 * 12, nchunks=12, **rows) == (27, 1, 8)
    assert parts_plan(V=16, G=15, npt=6, ngt=1, cols=36 * 13, nchunks=13, **rows) == (15, 1, 8)
    rows.update(strided=False)
    assert parts_plan(V=2, G=11, npt=9, ngt=1, cols=42 * 5, nchunks=5, **rows) == (11, 1, 8)


def test_few_columns():
    assert parts_plan(V=4, G=8, npt=2, ngt=1, cols=17) is None
    assert parts_plan(V=4, G=5, npt=84, ngt=1, cols=4) is None
    assert parts_plan(V=16, G=10, npt=112, ngt=1, cols=15) is None
    assert parts_plan(V=4, G=2, npt=63, ngt=1, cols=30, nchunks=2) is None
    assert parts_plan(V=8, G=5, npt=21, ngt=1, cols=30) is None
    assert parts_plan(V=8, G=5, npt=21, ngt=1, cols=30, wide=True) == (5, 1, 16)
    assert parts_plan(V=4, G=8, npt=2, ngt=1, cols=60) == (8, 1, 16)
    assert parts_plan(V=8, G=20, npt=69, ngt=2, cols=39) == (3, 8, 2)
    assert parts_plan(V=8, G=39, npt=4, ngt=3, cols=18, gpt=13, wide=True) == (39, 1, 16)
    assert parts_plan(V=8, G=58, npt=3, ngt=4, cols=13) == (58, 1, 16)
    assert parts_plan(V=1, G=712, npt=1, ngt=45, cols=30, gpt=16) == (178, 4, 4)
    assert parts_plan(V=4, G=114, npt=10, ngt=8, cols=89) == (15, 8, 2)


def test_groups_of_a_tile():
    assert groups_of_tile(33, 2, 300, 8, 4, 512) == 17
    assert groups_of_tile(129, 5, 117, 8, 4, 512) == 32     # 468 full tiles in a round, 585 even ones not
    assert groups_of_tile(129, 5, 100, 8, 4, 512) == 26
    assert groups_of_tile(129, 5, 400, 8, 4, 512) == 26
    assert groups_of_tile(36, 2, 300, 8, 4, 512) == 18      # (wavefronts of three groups, not four)
    for G in range(1, 700):
        for ug in (2, 4):
            ngt = -(-G // (8 * ug))
            for npt in (1, 100, 512 // ngt + 1):
                gpt = groups_of_tile(G, ngt, npt, 8, ug, 512)
                assert gpt <= 8 * ug and -(-G // gpt) == ngt
