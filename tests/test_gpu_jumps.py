"""Residues that a force throws whole periods of the fixed-point copies away
within a list period (half a period is 64 A here), where a wrapped difference
would look near: against what the FP64 oracle does.  A fixed residue and one
0.2 to 0.8 A from it, whose repulsion moves it by a period (128 A) or by 1,024
of them and a little more in the first step; in the next nine nothing acts.  In
one call and in two, and with a force evaluation between."""
import numpy as np
import pytest

from synth import RunParams
from synth.structures import System

from test_gpu_lane_order import P  # noqa: F401

pytestmark = pytest.mark.gpu

PERIOD = 128.0
SCHEDULES = ["plain", "batched"]


def kick_distance(move, p):
    """Distance at which the repulsion moves a residue by `move` in a step."""
    return (p.h / p.zeta * 6.0 * p.eps_l * p.sigma**6 / move) ** (1.0 / 7.0)


def system(x, bonds=(), natives=(), r0=()):
    b = np.asarray(bonds, np.int32).reshape(-1, 2)
    n = np.asarray(natives, np.int32).reshape(-1, 2)
    return System("jumps", np.asarray(x, float), np.array([0, len(x)], np.int64), np.zeros(1, np.uint32),
                  np.zeros(len(x), np.int32), b, np.asarray(r0[:len(b)], float), n, np.asarray(r0[len(b):], float),
                  np.array([1] + [0] * (len(x) - 1), np.uint8))


def steps(P, s, p, schedule, calls, forces=False):  # noqa: F811
    c = P.from_system(s, p, schedule=schedule, energy_every=0)
    out = []
    for n in calls:
        c.step(n)
        out.append(c.get_coordinates())
        if forces:
            out.append(c.compute_forces()[0])
    c.close()
    return out


# movement is checked step by step, or (long list periods with noise) by place
CHECKS = {"by step": dict(kBT=0.0), "by place": dict(kBT=0.03, list_every=100)}


@pytest.mark.parametrize("schedule", SCHEDULES)
@pytest.mark.parametrize("check", CHECKS)
@pytest.mark.parametrize("periods", [1, 2, 1024])
def test_list_pair(P, orc, periods, check, schedule):  # noqa: F811
    p = RunParams(**CHECKS[check])
    move = periods * PERIOD + 1.5
    s = system([[0.0, 0.0, 0.0], [kick_distance(move, p), 0.0, 0.0]])
    x1, F1, x2, F2 = steps(P, s, p, schedule, [1, 9], forces=True)
    o = orc.OracleSystem(s, p)
    x1o, x2o = o.run(s.x, 1)[0], o.run(s.x, 10)[0]
    assert abs(x1o[1, 0] - move) < 1.0
    assert np.abs(x1 - x1o).max() <= 1e-5 * move
    # at 128 A the repulsion is 3e-11
    assert np.abs(F1).max() <= 1e-9 and np.abs(F2).max() <= 1e-9
    assert np.abs((x2 - x1) - (x2o - x1o)).max() <= 1e-6
    assert np.array_equal(x2, steps(P, s, p, schedule, [10])[0])


@pytest.mark.parametrize("schedule", SCHEDULES)
@pytest.mark.parametrize("check", CHECKS)
def test_native_pair(P, orc, check, schedule):  # noqa: F811
    """The fixed residue's contact (at its distance, 6 A), thrown off by a third
    residue; a period and 0.5 A away its force is 1e-12 and less."""
    p = RunParams(**CHECKS[check])
    d = kick_distance(PERIOD + 0.5, p)
    s = system([[0.0, 0.0, 0.0], [6.0, 0.0, 0.0], [6.0 - d, 0.0, 0.0]], (), [[0, 1]], [6.0])
    x1, x2 = steps(P, s, p, schedule, [1, 9])
    o = orc.OracleSystem(s, p)
    x1o, x2o = o.run(s.x, 1)[0], o.run(s.x, 10)[0]
    assert np.abs(x2 - x2o).max() <= 1e-5 * PERIOD
    assert np.abs((x2 - x1) - (x2o - x1o)).max() <= 1e-6


@pytest.mark.parametrize("calls", [[2], [1, 1]])
@pytest.mark.parametrize("schedule", SCHEDULES)
def test_bond(P, orc, schedule, calls):  # noqa: F811
    """A bond stretched by a period is broken."""
    p = RunParams(kBT=0.0)
    d = kick_distance(PERIOD, p)
    s = system([[0.0, 0.0, 0.0], [3.8, 0.0, 0.0], [3.8 - d, 0.0, 0.0]], [[0, 1]], (), [3.8])
    assert orc.OracleSystem(s, p).run(s.x, 2)[3] != 0
    with pytest.raises(P.SopError) as e:
        steps(P, s, p, schedule, calls)
    assert e.value.name == "SOP_E_FENE"


def test_clash_in_a_box_of_particles(P, orc):  # noqa: F811
    """One clash among 300 free particles: the steps that follow it within the
    list period (all from the compensated positions, over several tiles)
    against the oracle, call by call bit for bit."""
    p = RunParams(kBT=0.0)
    i = np.arange(300)
    x = 4.6 * np.stack([i % 7, (i // 7) % 7, i // 49], 1) + 0.2 * np.random.default_rng(4).standard_normal((300, 3))
    x[150] = x[149] + np.array([kick_distance(40.0, p), 0.0, 0.0])
    s = system(x)
    a = steps(P, s, p, "plain", [25])[0]
    xo, _, _, st = orc.OracleSystem(s, p).run(s.x, 25)
    assert st == 0 and np.abs(xo[149] - x[149]).max() > 20.0
    assert np.abs(a - xo).max() <= 2e-4  # the kick itself, 40 A, to 2e-6
    assert np.array_equal(a, steps(P, s, p, "plain", [3, 4, 18])[-1])


@pytest.mark.parametrize("far", [4.0e4, 1024 * PERIOD + 3.9])
def test_wide_trajectory(P, orc, far):  # noqa: F811
    """Batched: pairs farther apart than half the 1,024 periods that the copies
    hold, native partners among them."""
    p = RunParams(kBT=0.0)
    x = np.array([[0.0, 0.0, 0.0], [3.9, 0.1, 0.0], [far, 0.0, 0.0], [far + 0.2, 4.0, 0.0]])
    s = system(x, (), [[0, 3], [1, 2]], [6.0, 6.0])
    o = orc.OracleSystem(s, p)
    c = P.from_system(s, p, schedule="batched")
    F = c.compute_forces()[0]
    assert np.abs(F - o.forces(x)[0]).max() <= 1e-5 * np.abs(o.forces(x)[0]).max()
    c.step(20)
    assert np.abs(c.get_coordinates() - o.run(x, 20)[0]).max() <= 1e-4
    c.close()


def test_non_finite_coordinates(P):  # noqa: F811
    """A coordinate beyond single precision is reported by either schedule."""
    s = system([[0.0, 0.0, 0.0], [1.0e39, 0.0, 0.0]])
    for schedule in SCHEDULES:
        c = P.from_system(s, RunParams(), schedule=schedule)
        with pytest.raises(P.SopError) as e:
            c.step(2)
            c.synchronize()
        assert e.value.name == "SOP_E_NONFINITE"
        c.close()
