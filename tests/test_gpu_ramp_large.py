"""Particle counts of the ramp model above what one launch of eight lanes a
particle holds (2^29 particles are 2^32 lanes), with noise: the first step of
particles on both sides of every launch's edge against the oracle's Gaussians."""
import math

import pytest

from test_gpu_ramp import KBT, KSP, RF, SEED, XI, env  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [2**28 + 1, 2**29 + 65])
def test_more_particles_than_one_launch_holds(env, M):  # noqa: F811
    torch, orc, P = env
    h = 25.0
    x = torch.zeros((M, 2), dtype=torch.float32, device="cuda")
    P.ramp_run(P.ramp_params(RF, XI, KSP, KBT, h, seed=SEED, stream=4), x, 0, 1, moments=False)
    sig = math.sqrt(2.0 * KBT * h / XI)
    for m in {0, 2**28 - 1, 2**28, 2**29 - 1, 2**29, M - 1}:
        if m < M:
            # single-precision Box-Muller: 6e-7 of the largest radius, 5.8
            assert abs(float(x[m, 0]) - sig * orc.gauss3(SEED, m, 4, 0)[0]) <= 4e-6 * sig, m
    assert int((x[:, 0] == 0.0).sum()) < 100  # every particle has moved
