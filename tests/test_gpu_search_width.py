"""The skin search at the tile counts where its workgroups change width (1,024
lanes up to 256 tiles, 512 up to 640, then 256), with more bonded and native
entries than a part keeps in registers, and with several windows of
candidates: lists bit-exact and forces against the FP64 oracle, and 30 steps
against direct launches of another tile size."""
import numpy as np
import pytest

from synth import RunParams
from synth.structures import _system, saw_batch

from parity import TRAJ_TOL, assert_forces, oracle_reference
from test_gpu_lane_order import P, manual, tiles  # noqa: F401

pytestmark = pytest.mark.gpu


def crowded(n):
    """n clusters of 48 residues, all natives of one another."""
    x = 4.3 * np.stack(np.meshgrid(range(4), range(4), range(3)), -1).reshape(-1, 3)
    i, j = np.triu_indices(48, 1)
    k = np.arange(n)
    o = np.stack([120.0 * (k % 9), 120.0 * (k // 9 % 9), 120.0 * (k // 81)], 1)
    nat = (np.stack([i, j], 1)[None] + 48 * k[:, None, None]).reshape(-1, 2)
    x = (x[None] + o[:, None]).reshape(-1, 3)
    return manual(x, (), nat, np.linalg.norm(x[nat[:, 0]] - x[nat[:, 1]], axis=1)), RunParams()


def dense(n):
    """n residues 3.6 A apart: more than 1,024 candidates around a tile."""
    m = int(np.ceil(n ** (1 / 3)))
    g = np.stack(np.meshgrid(range(m), range(m), range(m)), -1).reshape(-1, 3)[:n]
    return manual(3.6 * g), RunParams(r_list=12.0, list_capacity=512)


CASES = {"256 tiles": lambda: tiles(256), "257 tiles": lambda: tiles(257), "crowded 8": lambda: crowded(8),
         "crowded 400": lambda: crowded(400), "dense 3000": lambda: dense(3000), "dense 18000": lambda: dense(18000)}


@pytest.mark.parametrize("name", CASES)
def test_search_width(P, orc, name):  # noqa: F811
    s, p = CASES[name]()
    o = orc.OracleSystem(s, p)
    x = s.x + 0.05 * np.random.default_rng(3).standard_normal(s.x.shape)
    c = P.from_system(s, p, coordinates=x)
    ref = o.pairlist(x)
    Fo, _, _, S, _ = oracle_reference(o, x, pairs=ref)
    F, _, _ = c.compute_forces()
    assert np.array_equal(c.get_pairlist(), ref)
    assert_forces(F, Fo, S, name)
    got = []
    for q in (c, P.from_system(s, p, tile=128, graph_steps=0)):
        q.set_coordinates(x)
        q.step(30)
        got.append(q.get_coordinates())
        q.close()
    assert float(np.linalg.norm(got[0] - got[1], axis=1).max()) <= TRAJ_TOL
