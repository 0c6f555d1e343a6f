"""A context with long list periods makes no graph of ten of them: 10,000 steps
right after the 64 replays that would call for one take what the next 10,000
do (48 ms; 70 ms where a graph of 10,000 steps was made)."""
import time

import pytest

from synth import RunParams, make_config

from test_gpu_lane_order import P  # noqa: F401

pytestmark = pytest.mark.gpu


def test_long_list_periods_make_no_long_graph(P):  # noqa: F811
    c = P.from_system(make_config("c0"), RunParams(list_every=1000))
    c.step(65_000)
    c.synchronize()
    took = []
    for _ in range(3):
        t = time.perf_counter()
        c.step(10_000)
        c.synchronize()
        took.append(time.perf_counter() - t)
    print(took)
    assert took[0] <= 1.2 * min(took[1:])
    c.close()
