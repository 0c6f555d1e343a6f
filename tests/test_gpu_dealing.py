"""Which lane of a residue sums a partner, and so every bit of the forces,
depends on the list alone, also where one residue class of the skin rows is more
than a lane holds (24 partners here) and they are dealt in turn: 64 residues
whose ids are all multiples of 16 on a grid of 12 A, of which a list row holds
at most 18, a skin row at 4 A 26 and at 20 A up to 60; and at 8 A, where the
list rows themselves are dealt in turn.  Same bits at every skin, and the oracle."""
import numpy as np
import pytest

from synth import RunParams

from parity import assert_energies, assert_forces, oracle_reference
from test_gpu_lane_order import P, manual  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("edge", [8.0, 12.0])
def test_forces_do_not_depend_on_the_skin(P, orc, edge):  # noqa: F811
    n, g = 1024, np.arange(64)
    i = np.arange(n)
    x = np.stack([400.0 + 45.0 * (i % 10), 45.0 * ((i // 10) % 10), 45.0 * (i // 100)], 1)
    x[::16] = edge * np.stack([g % 4, (g // 4) % 4, g // 16], 1)
    x += 0.05 * np.random.default_rng(9).standard_normal(x.shape)
    s, p = manual(x), RunParams(list_capacity=64, eps_l=1.0e4, kBT=0.0)
    o = orc.OracleSystem(s, p)
    ref = o.pairlist(x)
    Fo, Eo, _, S, Em = oracle_reference(o, x, pairs=ref)
    got = []
    for skin in (0.0, 4.0, 8.0, 20.0):
        c = P.from_system(s, p)
        c.set_list_skin(skin)
        F, E, _ = c.compute_forces()
        assert np.array_equal(c.get_pairlist(), ref)
        c.set_coordinates(x)
        c.step(25)
        got.append((F, E, c.get_coordinates()))
        c.close()
    assert_forces(got[0][0], Fo, S, f"edge {edge}")
    assert_energies(got[0][1], Eo, Em, s.res_offsets, f"edge {edge}")
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert np.array_equal(a, b)
