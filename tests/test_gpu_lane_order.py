"""The plain schedule's work split and fixed-point positions where they can go
wrong, against the FP64 oracle: every lane count (the tile counts on both
sides of each change), positions across the wrap of the fixed-point copies,
bonded pairs in and out of their reach (and a whole period apart, where a
wrapped difference would look like a contact), tiles too long for one origin,
partners that would all fall to one lane, slot ids that need 32 bits, and
parameters for which the copies are too coarse.  The gates are those of every
force test: bit-exact lists, forces within 1e-5 of each residue's scale, and
20-step trajectories (two list rebuilds) within 1e-4 A.
"""
import numpy as np
import pytest

from synth import RunParams
from synth.structures import System, _system, saw_batch

from parity import TRAJ_TOL, assert_energies, assert_forces, oracle_reference

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_1003_1148_amd as P
    P.lib()
    return P


def manual(x, bonds=(), natives=(), native_r0=()):
    b = np.asarray(bonds, np.int32).reshape(-1, 2)
    n = np.asarray(natives, np.int32).reshape(-1, 2)
    return System("manual", np.asarray(x, float), np.array([0, len(x)], np.int64), np.zeros(1, np.uint32),
                  np.zeros(len(x), np.int32), b, np.linalg.norm(x[b[:, 0]] - x[b[:, 1]], axis=1), n,
                  np.asarray(native_r0, float))


def tiles(n):
    """n tiles of one 40-residue chain each."""
    w = saw_batch(np.full(8, 40), np.random.default_rng(5))
    return _system("tiles", [[w[t % 8]] for t in range(n)]), RunParams()


def shifted(v):
    w = saw_batch(np.array([300]), np.random.default_rng(6))[0]
    return _system("shifted", [[w - w[150] + np.asarray(v)]]), RunParams()


def apart(d):
    """Two chains whose like residues are natives of 6 A, d apart along x."""
    w = saw_batch(np.array([40]), np.random.default_rng(7))[0]
    x = np.concatenate([w, w + np.array([d, 0.3, -0.2])])
    k = np.arange(39)
    bonds = np.concatenate([np.stack([k, k + 1], 1), np.stack([k + 40, k + 41], 1)])
    nat = np.stack([np.arange(0, 40, 3), np.arange(0, 40, 3) + 40], 1)
    return manual(x, bonds, nat, np.full(len(nat), 6.0)), RunParams()


def straight():
    """A chain pulled straight: 64 residues span 243 A."""
    rng = np.random.default_rng(8)
    x = np.stack([3.8 * np.arange(200), np.zeros(200), np.zeros(200)], 1) + 0.1 * rng.standard_normal((200, 3))
    return _system("straight", [[x]]), RunParams()


def one_class():
    """56 residues in contact whose ids are all multiples of 16, the rest 22 A apart."""
    n = 16 * 56
    i = np.arange(n)
    x = np.stack([300.0 + 22.0 * (i % 10), 22.0 * ((i // 10) % 10), 22.0 * (i // 100)], 1)
    g = np.arange(56)
    x[::16] = 3.9 * np.stack([g % 4, (g // 4) % 4, g // 16], 1)
    return manual(x + 0.05 * np.random.default_rng(9).standard_normal(x.shape)), RunParams(list_capacity=64)


def wide_ids():
    """A compact tile with partners 69,900 ids away."""
    n = 70_000
    i = np.arange(n)
    x = np.stack([2000.0 + 60.0 * (i % 42), 60.0 * ((i // 42) % 42), 60.0 * (i // 1764)], 1)
    c = np.concatenate([np.arange(64), np.arange(n - 48, n)])
    g = np.arange(len(c))
    x[c] = 4.4 * np.stack([g % 5, (g // 5) % 5, g // 25], 1)
    return manual(x), RunParams()


def coarse_list():
    s, _ = shifted((0.0, 0.0, 0.0))
    return s, RunParams(sigma=0.01, eps_l=1e12)


def coarse_bonds():
    s, _ = shifted((0.0, 0.0, 0.0))
    s.natives = np.concatenate([s.natives, [[0, 299]]]).astype(np.int32)
    s.native_r0 = np.append(s.native_r0, 0.2)
    return s, RunParams()


CASES = {
    "1 tile": lambda: tiles(1), "200 tiles": lambda: tiles(200), "201 tiles": lambda: tiles(201),
    "640 tiles": lambda: tiles(640), "641 tiles": lambda: tiles(641),
    "wrap at 64": lambda: shifted((63.99, -64.01, 64.0)), "wrap at 128": lambda: shifted((-128.0, 127.9, 191.9)),
    "1e5 A": lambda: shifted((1.0e5, -2.5e4, 7.7e4)),
    "in reach": lambda: apart(31.0), "out of reach": lambda: apart(33.0), "a period apart": lambda: apart(134.0),
    "two periods apart": lambda: apart(-251.0), "straight": straight, "one class": one_class,
    "wide ids": wide_ids, "coarse list": coarse_list, "coarse bonds": coarse_bonds,
}


@pytest.mark.parametrize("name", CASES)
def test_lane_order(P, orc, name):
    s, p = CASES[name]()
    o = orc.OracleSystem(s, p)
    rng = np.random.default_rng(3)
    x = s.x + 0.05 * rng.standard_normal(s.x.shape)
    c = P.from_system(s, p, coordinates=x)
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
