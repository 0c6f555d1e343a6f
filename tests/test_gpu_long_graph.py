"""Graphs of several list periods, which a context makes once it has replayed
its short ones 64 times: positions and energy records bit for bit those of
direct launches, with and without records, across calls that end inside a
period, an odd number of steps a period, and the underdamped integrator."""
import numpy as np
import pytest

from synth import RunParams
from synth.structures import _system, saw_batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("graph_steps", [1, 3])
@pytest.mark.parametrize("every, L, underdamped", [(0, 10, False), (100, 10, False), (210, 7, False), (300, 10, True)])
def test_long_graphs(every, L, underdamped, graph_steps):
    import torch
    import paper_1003_1148_amd as P
    assert torch.cuda.is_available()
    w = saw_batch(np.array([90, 41]), np.random.default_rng(12))
    s = _system("graphs", [[v] for v in w])
    got = []
    for g in (0, graph_steps):
        c = P.from_system(s, RunParams(list_every=L), graph_steps=g, energy_every=every)
        if underdamped:
            c.set_integrator("underdamped", mass=5.0)
        rec = []
        for n in (64 * L * graph_steps + 3, 211, 400, 5):
            c.step(n)
            rec += [c.get_coordinates(), *(c.get_energies() if every else ())]
        got.append(rec)
        c.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b)
