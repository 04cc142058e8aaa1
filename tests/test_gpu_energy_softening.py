"""The FP64 energy with softenings that its fast inverse root does not take: an
infinite one gives every pair the weight 0 (the energy is the kinetic one), a
zero or negative one and a NaN go through the square root and the division; and
the ends of the fast form's range.  Tolerance as test_gpu_energy.py: 1e-11 of
the sum of magnitudes."""
import numpy as np
import pytest

import oracle
from gpu_helpers import gpu_view, say

import paper_2302_08251_amd as lm
from paper_2302_08251_amd import synth

pytestmark = pytest.mark.gpu

REC = ["f32"] * 7


@pytest.mark.parametrize("n", [2, 65, 300, 1000])
def test_softening_values(n):
    planes = synth.particles(n, 3, dtype=np.float32)
    v = gpu_view(REC, {"kind": "soa_mb"}, n, oracle.store_planes(REC, {"kind": "soa_mb"}, planes))
    pos = np.stack(planes[0:3], 1).astype(np.float64)
    vel = np.stack(planes[3:6], 1).astype(np.float64)
    m = planes[6].astype(np.float64)
    kin = 0.5 * float((m * (vel * vel).sum(1)).sum())
    say("infinite softening", n)
    assert abs(lm.nbody_energy(v, np.inf) - kin) <= 1e-11 * kin
    for eps2 in (0.0, float(np.float32(1e-45)), float(np.finfo(np.float32).max)):
        ref = oracle.energy(pos, vel, m, eps2)
        say("softening", n, eps2, ref)
        assert abs(lm.nbody_energy(v, eps2) - ref) <= 1e-11 * (kin + abs(ref - kin))
    assert np.isnan(lm.nbody_energy(v, np.nan))
    assert np.isnan(lm.nbody_energy(v, -1e30))
