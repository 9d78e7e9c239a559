"""The kernels that walk chunks of channels: which launches give a wavefront one group, or a part of one
(csrc/alcs_parts_plan.h)."""
import math
import random

from parts_plan import parts_plan


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
