"""Meshes with more than 65 536 cells along one axis: indices that take more
than 16 bits, through every form of the step, against the FP64 oracle.

One sort and six steps, so the cells are those of the given positions.  A
position difference of d chamber lengths shifts a cloud-in-cell weight by up
to 70 000 d, and d stays below 1e-13 in six steps: a node's density agrees
within 1e-8 of the largest one.  Two forms of the step hold the same
positions and add the same terms: within 1e-12.
"""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import assert_state_close, assert_tallies_equal, boosted, gpu_run, oracle
from test_gpu_period import STATE

pytestmark = pytest.mark.gpu

AXES = {"x": (70_001, 3, 2), "y": (2, 70_001, 3), "z": (3, 2, 70_001), "z_alone": (1, 1, 70_001)}


def thin(axis, fields, n=3_001):
    mesh = AXES[axis]
    p = boosted(W.base_params(n, *mesh, seed=31))
    p.update(weight=5e7, deposit_mask=fields, sort_every=9)
    st = W.random_state(p, seed=8, q_max=8, v_ev=300.0, frac_atoms=0.15, radius_frac=0.99, birth_max=2)
    # 600 particles in one cell beyond index 65 536, on the axis otherwise
    rng = np.random.default_rng(9)
    h = (2 * p["R0"] / mesh[0], 2 * p["R0"] / mesh[1], p["L"] / mesh[2])
    low = (-p["R0"], -p["R0"], -p["L"] / 2)
    for c, k in enumerate("xyz"):
        cell = 65_900 if mesh[c] > 65_536 else mesh[c] // 2
        st[k][:600] = low[c] + (cell + 0.1 + 0.8 * rng.random(600)) * h[c]
    return p, st


@pytest.mark.parametrize("fields", [3, 15])
@pytest.mark.parametrize("axis", list(AXES))
def test_indices_beyond_16_bits(axis, fields):
    p, st = thin(axis, fields)
    forms = {"launch": (dict(events=True), (6,)), "single": (dict(events=True), (1,) * 6),
             "split": (dict(events=True, split=True), (6,))}
    runs = {}
    for name, (options, calls) in forms.items():
        r = gpu_run(p, **options)
        r.set_state(st, step=3)
        for k in calls:
            r.step(k)
        runs[name] = r
    o = oracle(p)
    o.set_state(st, step=3)
    o.step(6)
    a = runs["launch"].get_state()
    assert_state_close(a, o.get_state(), p, what=axis, tol=1e-11)
    for name, r in runs.items():
        b = r.get_state()
        for k in STATE:
            assert np.array_equal(a[k], b[k]), (name, k)
        assert np.array_equal(r.events(), o.events())
        assert_tallies_equal(r.tallies(), o.tallies(), name)
        for f in range(4):
            if fields >> f & 1:
                d, l, e = r.density(f)[0], runs["launch"].density(f)[0], o.density(f)[0]
                assert np.abs(d - e).max() <= 1e-8 * np.abs(e).max(), (name, f)
                assert np.abs(d - l).max() <= 1e-12 * max(1.0, np.abs(l).max()), (name, f)
