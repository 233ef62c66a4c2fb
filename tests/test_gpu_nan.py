"""A collision probability that is not a number (an ion whose velocity is
not): the ionisation channels before it are decided as the oracle decides
them.  Many ions, since a decision on less than the whole uniform differs
for a few in a hundred thousand steps only.
"""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import gpu_run, oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("calls", [(8,), (1,) * 8])
@pytest.mark.parametrize("extended", [False, True])
def test_decisions_beside_a_probability_that_is_not_a_number(extended, calls):
    p = W.base_params(300_007, 16, 16, 32, seed=31)
    gas = W.argon(n0_m3=1e13, outside_rates=True)
    p["species"] = [W.with_extended_mcc(gas) if extended else gas]
    # no push and no pools: the positions stay, the velocities touch nothing else
    p.update(process_mask=W.P_IONIZE | W.P_CX | (W.P_ELASTIC if extended else 0), sort_every=50, dt=5e-7, ne_out=1e18)
    st = W.random_state(p, seed=8, q_max=6, v_ev=300.0, frac_atoms=0.1, radius_frac=0.9, birth_max=2)
    st["vx"] = np.full_like(st["vx"], np.nan)
    g, o = gpu_run(p, events=True), oracle(p)
    for r in (g, o):
        r.set_state(st, step=3)
    for k in calls:
        g.step(k)
    o.step(8)
    a, b = g.get_state(), o.get_state()
    assert (b["q"] != st["q"]).sum() > 10_000  # the channels fire
    for k in ("q", "birth"):
        assert np.array_equal(a[k], b[k]), k
    assert np.array_equal(g.events(), o.events())
