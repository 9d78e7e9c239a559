"""Launches that fill the chip, with group counts that are no multiple of what the workgroups hold: the groups are dealt
evenly to the group tiles and to their wavefronts (3x3, and 1x1 kernels that walk chunks of channels)."""
import pytest

import workloads
from gpu_util import TOL, oracle_ref, rel_err, run_sparse

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
