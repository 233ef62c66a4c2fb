"""Runs with cell grids, with three of them in turn and with two, however the
steps are launched: one by one, by captured periods (of a length that leaves
the grids in any of their places), in a batch, after a state set anew.

The grids hold whole numbers, so all forms agree bit for bit, and with the
oracle in every count.
"""
import numpy as np
import pytest

import workloads as W
from test_gpu_parity import assert_tallies_equal, boosted, gpu_run, oracle
from test_gpu_period import STATE

pytestmark = pytest.mark.gpu

MODELS = {"ne": dict(self_ne=True), "n0": dict(self_n0=True), "both": dict(self_ne=True, self_n0=True),
          "partners": dict(self_ne=True, self_n0=True, cx_partner=True)}


@pytest.mark.parametrize("every", [1, 3, 4, 5])
@pytest.mark.parametrize("n", [601, 30_011])  # 8192 cells: two grids, three grids
@pytest.mark.parametrize("model", list(MODELS))
def test_forms_of_a_run_with_cell_grids(model, n, every):
    import torch

    import paper_1507_03392_amd as ecr
    p = boosted(W.base_params(n, 16, 16, 32, seed=31))
    p.update(weight=5e7, sort_every=every, process_mask=W.P_ALL | W.P_HEAT, **MODELS[model])
    st = W.random_state(p, seed=8, q_max=8, v_ev=300.0, frac_atoms=0.3, radius_frac=0.99, birth_max=2)
    stream = torch.cuda.Stream()
    first, steps = 4 * every, 17
    runs = {}
    for form in ("one by one", "graph", "batch", "again"):
        r = gpu_run(p, stream=stream)
        if form == "again":
            r.set_state(st, step=first)
            r.step(2)
        r.set_state(st, step=first)
        if form == "graph":
            r.step(every)
            for k in (steps - every - 2, 2):
                r.step_graph(k)
        elif form == "batch":
            other = gpu_run(W.with_(p, self_ne=False, self_n0=False, cx_partner=False), stream=stream)
            other.set_state(st, step=first)
            for k in (every, steps - every):
                ecr.step_batch([r, other], k, stream)
        else:
            for _ in range(steps):
                r.step(1)
        runs[form] = r
    a = runs["one by one"].get_state()
    for form, r in runs.items():
        b = r.get_state()
        assert b["step"] == first + steps
        for k in STATE:
            assert np.array_equal(a[k], b[k]), (form, k)
        assert_tallies_equal(runs["one by one"].tallies(), r.tallies(), form)
    o = oracle(p)
    o.set_state(st, step=first)
    o.step(steps)
    assert_tallies_equal(runs["graph"].tallies(), o.tallies(), "oracle")
