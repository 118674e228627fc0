"""Expansions that outgrow what they were sized for, against the oracle: a
first step whose ball overfills the hash table and the rows (the table is
left while it fills and the step repeated with a larger one), and runs long
under a state cap far below the ball of their selection (the rounds stop as
soon as the rows found exceed the cap, in place and from scratch).  Sets bit
for bit; amplitudes with the element bound of gpu_helpers."""
import numpy as np
import pytest

import paper_2603_07341_amd as P
from oracle import oracle as O
from tests.gpu_helpers import assert_amps, assert_same_set, sort_rows
import workloads as WL

pytestmark = pytest.mark.gpu


def pair(name, run_over, warm=1, **over):
    cfg = dict(WL.CONFIGS[name], **over)
    p = WL.model_params(cfg)
    run = dict(WL.run_params(cfg), **run_over)
    init = WL.initial_state(cfg)
    gs = P.Sim(P.Model(p), run, *init)
    gs.set_tuning(warm=warm)
    return gs, O.Sim(O.Model(p), run, *init)


def compare(gs, os_, steps):
    for which in (O.SET_M, O.SET_S):
        assert_same_set(gs.get_set(which), os_.get_set(which), "set %d" % which)
    gk, ga = sort_rows(*gs.state())
    ok, oa = os_.state()
    assert np.array_equal(gk, ok)
    assert_amps(ga, oa, 1e-10, steps=steps)


@pytest.mark.parametrize("k_init", [6, 7, 8])
def test_first_ball_overfills_the_table(k_init):
    # balls of 2.5e4 to 4e5 rows from one row, in a table sized for 65537
    gs, os_ = pair("cube4", {}, extent=[3, 3, 3], max_states=0, precision=64,
                   eps_sigma=0.05, eps_seed=3, k_init=k_init)
    gs.step(1)
    os_.step(1)
    compare(gs, os_, 1)


@pytest.mark.parametrize("warm", [0, 1, 2])
@pytest.mark.parametrize("cap", [500, 3000])
def test_cap_far_below_the_ball(cap, warm):
    gs, os_ = pair("ring12", dict(max_states=cap), warm, extent=[6, 1, 1],
                   cutoff=[6], theta=1e-9, k=3, k_init=3)
    for step in range(24):
        gs.step(1)
        os_.step(1)
        assert gs.observe()["n_S"] <= cap
        compare(gs, os_, step + 1)
