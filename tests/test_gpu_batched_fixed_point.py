"""The batched schedule's fixed-point positions where they can go wrong, against
the FP64 oracle: positions across the wrap of the copies, bonded pairs in and
out of the reach of plain differences (and whole periods apart, where a
wrapped difference would look like a contact), rows that end anywhere in an
eight, residues with more bonded entries than the workgroup keeps in LDS, and
parameters for which the copies are too coarse or the period too short for the
list.  Gates as in every force test.  Farther out than the direct conversion
reaches, forces keep the bits that they have at the origin."""
import numpy as np
import pytest

from synth import RunParams
from synth.structures import _system, saw_batch

from parity import TRAJ_TOL, assert_energies, assert_forces, oracle_reference
from test_gpu_lane_order import P, apart, coarse_bonds, coarse_list, manual, shifted, straight  # noqa: F401

pytestmark = pytest.mark.gpu


def row_ends():
    """Chains of 4 to 43 residues, 2.5 A apart: rows of 0 to 39 partners."""
    w = saw_batch(np.full(1, 43), np.random.default_rng(4))[0]
    return _system("rows", [[0.55 * w[:m]] for m in range(4, 44)]), RunParams()


def crowded():
    """24 residues that are all natives of one another: 23 entries each."""
    x = 4.2 * np.stack(np.meshgrid(range(4), range(3), range(2)), -1).reshape(-1, 3)
    x = np.concatenate([x + np.array([500.0 * g, 0, 0]) for g in range(10)])
    i, j = np.triu_indices(24, 1)
    n = np.concatenate([np.stack([i, j], 1) + 24 * g for g in range(10)])
    return manual(x, (), n, np.linalg.norm(x[n[:, 0]] - x[n[:, 1]], axis=1)), RunParams()


CASES = {
    "wrap at 64": lambda: shifted((63.99, -64.01, 64.0)), "wrap at 128": lambda: shifted((-128.0, 127.9, 191.9)),
    "1e5 A": lambda: shifted((1.0e5, -2.5e4, 7.7e4)),
    "in reach": lambda: apart(31.0), "out of reach": lambda: apart(33.0), "a period apart": lambda: apart(134.0),
    "two periods apart": lambda: apart(-251.0), "straight": straight, "coarse list": coarse_list,
    "short period": coarse_bonds, "row ends": row_ends, "crowded": crowded,
}


@pytest.mark.parametrize("wg", [256, 512, 1024])
@pytest.mark.parametrize("name", CASES)
def test_batched_fixed_point(P, orc, name, wg):  # noqa: F811
    s, p = CASES[name]()
    n = int(np.diff(s.res_offsets).max())
    if n > wg:
        pytest.skip("longer than the workgroup")
    o = orc.OracleSystem(s, p)
    x = s.x + 0.05 * np.random.default_rng(3).standard_normal(s.x.shape)
    c = P.from_system(s, p, coordinates=x, schedule="batched", batch=(wg, 20))
    ref = o.pairlist(x)
    Fo, Eo, _, S, Em = oracle_reference(o, x, pairs=ref)
    F, E, _ = c.compute_forces()
    assert np.array_equal(c.get_pairlist(), ref)
    assert_forces(F, Fo, S, name)
    assert_energies(E, Eo, Em, s.res_offsets, name)
    c.set_coordinates(x)
    c.step(20)
    xo, _, _, st = o.run(x, 20)
    assert st == 0
    assert float(np.linalg.norm(c.get_coordinates() - xo, axis=1).max()) <= TRAJ_TOL
    c.close()


@pytest.mark.parametrize("d", [2.0**29, -(2.0**29)])
def test_beyond_the_direct_conversion(P, d):  # noqa: F811
    """12 residues 2^29 A out, with r_list 200 A (the lists, taken from high
    parts 64 A apart there, hold every pair at both places): the coordinates
    are exact, so the forces are those at the origin bit for bit."""
    w = saw_batch(np.array([12]), np.random.default_rng(6))[0]
    w = np.round(w * 2.0**12) / 2.0**12
    s = _system("far", [[w]])
    F = []
    for x in (w, w + d):
        c = P.from_system(s, RunParams(r_list=200.0), coordinates=x, schedule="batched")
        F.append(c.compute_forces()[0])
        assert len(c.get_pairlist()) > 40
        c.close()
    assert np.array_equal(F[0], F[1])


@pytest.mark.parametrize("wg", [256, 1024])
@pytest.mark.parametrize("every", [15, 16, 17, 40])
def test_record_launches(P, every, wg):  # noqa: F811
    """Energy intervals around the one from which a record step is a launch of
    its own: positions and the last record bit for bit those of one step a
    call on the other workgroup size."""
    w = saw_batch(np.array([170, 60, 33]), np.random.default_rng(11))
    s = _system("records", [[v] for v in w])
    got = []
    for wg_, calls in ((wg, [7, 43, 6]), (1280 - wg, [1] * 56)):
        c = P.from_system(s, RunParams(), schedule="batched", batch=(wg_, 20), energy_every=every)
        for n in calls:
            c.step(n)
        got.append((c.get_coordinates(), *c.get_energies()))
        c.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("packs", [512, 513])
def test_one_and_two_lanes_a_residue(P, packs):  # noqa: F811
    """Packs of 256 on both sides of the count up to which two lanes serve a
    residue, against the first 12 chains alone (two lanes) on packs of 512
    (one): bit for bit."""
    w = saw_batch(np.full(12, 150), np.random.default_rng(13))
    got = []
    for n, wg in ((packs, 256), (12, 256), (12, 512)):
        s = _system("lanes", [[w[t % 12]] for t in range(n)])
        c = P.from_system(s, RunParams(), schedule="batched", batch=(wg, 25))
        c.step(25)
        got.append(c.get_coordinates()[:12 * 150])
        c.close()
    assert np.array_equal(got[0], got[1])
    assert np.array_equal(got[0], got[2])
