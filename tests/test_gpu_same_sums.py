"""The momentum and energy sums of the collisions come out the same, bit for
bit, from one run to the next: which workgroup takes which chunk and the order
of what it adds are fixed.  Sparse, populous and crowded cells, one and
several steps a launch, one chunk, pairs of chunks, pairs and a rest of single
ones, and groups of them to a workgroup; and all of these against the launches
of several steps, which take one chunk.

Summed in another order, 5 million positive terms agree within 1e-11 (their
rounding adds up like a random walk, to some 1e-13).
"""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import assert_tallies_equal, boosted, gpu_run
from test_gpu_period import STATE, crowd

pytestmark = pytest.mark.gpu

SUMS = ("coul_dp", "coul_de", "coul_e")
CASES = {
    # n, mesh, radius of the ions (the share of the chamber's cells they fill), crowded cells
    "small": (3_001, (9, 9, 17), 0.99, ()),
    "dense": (40_009, (16, 16, 32), 0.33, (513, 1024, 1025, 3000)),
    "pairs": (470_003, (41, 40, 80), 0.99, (600, 1024, 2049)),
    "groups": (600_011, (32, 32, 64), 0.34, (700,)),
    "chunks of one cell": (460_007, (16, 16, 128), 0.35, ()),
    "pairs and single chunks": (1_010_003, (40, 40, 80), 0.99, (600,)),
}


def make(name, prec):
    n, mesh, radius, sizes = CASES[name]
    p = boosted(W.base_params(n, *mesh, seed=31))
    p.update(weight=5e7, precision=prec, sort_every=50)
    st = W.random_state(p, seed=8, q_max=8, v_ev=300.0, frac_atoms=0.1, radius_frac=radius, birth_max=2)
    crowd(p, st, sizes, 9)
    return p, st


@pytest.mark.parametrize("prec", [W.PREC_FP64, W.PREC_FP32])
@pytest.mark.parametrize("name", list(CASES))
def test_collision_sums_are_the_same_from_run_to_run(name, prec):
    p, st = make(name, prec)
    got = {}
    for calls in ((8,), (1,) * 8):
        for _ in range(3):
            r = gpu_run(p)
            r.set_state(st, step=3)
            for k in calls:
                r.step(k)
            got.setdefault(len(calls), []).append((r.tallies(), r.get_state(), [r.density(f)[0] for f in range(2)]))
    for runs in got.values():
        for t, s, _ in runs[1:]:
            for k in SUMS:
                assert np.array_equal(t[k], runs[0][0][k]), k
    (ta, sa, da), (tb, sb, db) = got[1][0], got[8][0]
    for k in STATE:
        assert np.array_equal(sa[k], sb[k]), k
    assert_tallies_equal(ta, tb, name)
    assert ta["coul_e"] == pytest.approx(tb["coul_e"], rel=1e-11)
    for a, b in zip(da, db):
        assert np.abs(a - b).max() <= 1e-12 * max(1.0, np.abs(b).max())
