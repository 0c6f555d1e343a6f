"""The plain schedule at list cutoffs from 5 to 50 A, against the FP64 oracle.
The period of the fixed-point copies follows the cutoff and the thermal drift
(half a period is 32 A up to 10.5 A, 64 A from 12 to 23, 256 A at 50; at zero
temperature 16 A at 5 and 32 A at 12), while a tile may reach 40 A from its
middle: positions relative to it must not wrap.  A globule of
1,000 residues (tiles 25 to 40 A in half-width) beside a helix that rises 1.1 A
a residue (64 of them span 70 A).  Gates as in every force test."""
import numpy as np
import pytest

from synth import RunParams, make_config
from synth.structures import _system

from parity import TRAJ_TOL, assert_energies, assert_forces, oracle_reference
from test_gpu_lane_order import P  # noqa: F401

pytestmark = pytest.mark.gpu


def globule_and_helix():
    k = np.arange(256)
    a = np.deg2rad(100.0 * k)
    helix = np.stack([2.375 * np.cos(a), 2.375 * np.sin(a), 1.1 * k], 1)
    return _system("cutoffs", [[make_config("c1").x], [helix]])


@pytest.mark.parametrize("tile", [64, 128, 256])
@pytest.mark.parametrize("r_list, kBT", [(5.0, None), (5.0, 0.0), (8.0, None), (10.0, None), (10.5, None),
                                         (12.0, None), (12.0, 0.0), (23.0, None), (50.0, None)])
def test_list_cutoffs(P, orc, r_list, kBT, tile):  # noqa: F811
    s = globule_and_helix()
    p = RunParams(r_list=r_list) if kBT is None else RunParams(r_list=r_list, kBT=kBT)
    o = orc.OracleSystem(s, p)
    x = s.x + 0.05 * np.random.default_rng(3).standard_normal(s.x.shape)
    c = P.from_system(s, p, coordinates=x, tile=tile)
    ref = o.pairlist(x)
    Fo, Eo, _, S, Em = oracle_reference(o, x, pairs=ref)
    F, E, _ = c.compute_forces()
    assert np.array_equal(c.get_pairlist(), ref)
    assert_forces(F, Fo, S, f"r_list {r_list} tile {tile}")
    assert_energies(E, Eo, Em, s.res_offsets, f"r_list {r_list} tile {tile}")
    c.set_coordinates(x)
    c.step(20)
    xo, _, _, st = o.run(x, 20)
    assert st == 0
    assert float(np.linalg.norm(c.get_coordinates() - xo, axis=1).max()) <= TRAJ_TOL
    c.close()
