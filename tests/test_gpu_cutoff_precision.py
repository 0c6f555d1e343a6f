"""The accuracy of bonded and native forces does not follow the list cutoff,
although the unit of the fixed-point copies does (3e-8 A at 20 A, 1.2e-7 A at 50 A
if nothing else held it).  Rounding a 3.8 A length to single precision is
2.4e-7 / sqrt(12) = 6.9e-8 A; two ends of unit u add u / sqrt(6), 1.5% to that at
3e-8 A and 22% at 1.2e-7 A: the L2 error at every cutoff is held to within 5% of
the one at 12 A."""
import numpy as np
import pytest

from synth import RunParams, make_config
from synth.structures import _system, saw_batch

from test_gpu_lane_order import P  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("schedule", ["plain", "batched"])
def test_force_error_does_not_grow_with_the_cutoff(P, orc, schedule):  # noqa: F811
    w = saw_batch(np.array([300, 200]), np.random.default_rng(50))
    s = _system("precision", [[make_config("c1").x], [w[0]], [w[1]]])
    x = s.x + 0.15 * np.random.default_rng(0).standard_normal(s.x.shape)
    err = {}
    for r in (12.0, 20.0, 24.0, 30.0, 50.0, 80.0, 200.0):
        p = RunParams(r_list=r, list_capacity=1024)
        Fo = orc.OracleSystem(s, p).forces(x)[0]
        c = P.from_system(s, p, coordinates=x, schedule=schedule)
        F = c.compute_forces()[0]
        c.close()
        err[r] = float(np.linalg.norm(F - Fo) / np.linalg.norm(Fo))
    print(err)
    assert max(err.values()) <= 1.05 * err[12.0]
