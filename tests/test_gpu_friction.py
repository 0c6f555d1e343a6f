"""The fixed-point copies with the underdamped integrator.  Their unit follows how
far residues drift in a list period: at low friction that is a flight at the
thermal velocity, not the overdamped drift, which grows without bound.  The
integrator may change anywhere in a list period, and with it the unit."""
import numpy as np
import pytest

from synth import RunParams, make_config

from parity import TRAJ_TOL
from test_gpu_lane_order import P  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("zeta", [1e-2, 1e-4, 1e-6])
def test_force_error_at_low_friction(P, orc, zeta):  # noqa: F811
    """List forces alone (no bonds, 5 A apart), 8 dr / r of a pair's force: the
    unit of overdamped drift would be 2e-6 A at 1e-4, that of flight is 3e-8 A,
    as at any friction of the overdamped integrator's use."""
    i = np.arange(512)
    x = 5.0 * np.stack([i % 8, (i // 8) % 8, i // 64], 1) + 0.3 * np.random.default_rng(5).standard_normal((512, 3))
    s = make_config("c1")
    s.x, s.res_offsets = x, np.array([0, 512], np.int64)
    s.bonds, s.bond_r0, s.natives, s.native_r0 = s.bonds[:0], s.bond_r0[:0], s.natives[:0], s.native_r0[:0]
    s.fixed, s.pulls, s.chain_id = None, [], s.chain_id[:512]
    err = []
    for p, mass in ((RunParams(h=0.01), None), (RunParams(h=0.01, zeta=zeta), 1.0)):
        c = P.from_system(s, p)
        if mass:
            c.set_integrator("underdamped", mass=mass)
        F = c.compute_forces()[0]
        c.close()
        Fo = orc.OracleSystem(s, p).forces(x)[0]
        err.append(float(np.linalg.norm(F - Fo) / np.linalg.norm(Fo)))
    print(err)
    assert err[1] <= 1.02 * err[0]


@pytest.mark.parametrize("first", ["overdamped", "underdamped"])
@pytest.mark.parametrize("at", [3, 10, 19])
def test_integrator_changes_within_a_list_period(P, orc, at, first):  # noqa: F811
    """zeta 0.5: half a period is 128 A for the one integrator, 64 A for the other."""
    s = make_config("c0")
    p = RunParams(zeta=0.5, h=0.01)
    o = orc.OracleSystem(s, p)
    c = P.from_system(s, p)
    zero = np.zeros_like(s.x)
    if first == "underdamped":
        c.set_integrator("underdamped", mass=1.0)
        xo = o.run_underdamped(s.x, zero, at, 1.0)[0]
        c.step(at)
        c.set_integrator("overdamped")
        xo = o.run(xo, 30 - at, step0=at)[0]
    else:
        xo = o.run(s.x, at)[0]
        c.step(at)
        c.set_integrator("underdamped", mass=1.0)
        xo = o.run_underdamped(xo, zero, 30 - at, 1.0, step0=at)[0]
    c.step(30 - at)
    d = float(np.abs(c.get_coordinates() - xo).max())
    print(d)
    assert d <= TRAJ_TOL
    c.close()
