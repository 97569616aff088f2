"""A launch shape set by itself leaves the rollout as it was, to the bit; setting
what get_tuning reports changes nothing."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

CASES = {"circles": lambda: W.c2("circles", K=3001, T=77, iters=1),
         "costmap": lambda: W.c2("costmap", K=700, T=40, iters=1),
         "quadrotor": lambda: W.c3(K=2100, T=30), "integrator": lambda: W.c1(K=40000, T=20)}


@pytest.mark.parametrize("name", sorted(CASES))
def test_other_fields_leave_the_rollout(name):
    import paper_2409_07563_amd as mppi
    ctl = mppi.Controller(CASES[name]())
    first, tuning = None, ctl.tuning()
    for shape in (None, {}, {"noise_calls": 2}, {"update_form": 0}, tuning):
        if shape is not None:
            ctl.set_tuning(**shape)
        ctl.set_iteration(0)
        ctl.sample()
        ctl.rollout()
        S = ctl.costs().cpu().numpy().view(np.uint32)
        first = S if first is None else first
        assert np.array_equal(S, first), shape
    assert ctl.tuning() == tuning
    ctl.close()
