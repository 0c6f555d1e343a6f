"""sop_step_timed on the batched schedule makes the launches that sop_step
makes: a record step from an interval of 16 on is one of its own.  Taken with
the steps around it, it costs all of them 15% and more (200 chains: 14.2 against
11.8 us a step at an interval of 100); alone 3%."""
import numpy as np
import pytest

from synth import RunParams, make_config

from test_gpu_lane_order import P  # noqa: F401

pytestmark = pytest.mark.gpu


def test_record_steps_are_timed_as_they_are_stepped(P):  # noqa: F811
    s = make_config("c3", n_traj=200)
    ctx = [P.from_system(s, RunParams(), schedule="batched", energy_every=E) for E in (0, 100)]
    for c in ctx:
        c.step_timed(200)
    ms = [[c.step_timed(400)[0] for _ in range(5)] for c in ctx]
    print(ms)
    assert min(ms[0]) > 0.0
    assert min(ms[1]) <= 1.09 * min(ms[0])
    for c in ctx:
        c.step_timed(1)  # step 2,200 is recorded
    assert ctx[1].get_energies()[1] == 2200
    assert np.array_equal(ctx[0].get_coordinates(), ctx[1].get_coordinates())
    for c in ctx:
        c.close()
