"""The FP64 energy of the n-body consumer against the oracle at the edges of
its blocks and runs (256 i-particles, runs of 64 j-particles and more), and
with values that its fast inverse root leaves to the plain form: an infinite
position (its pairs weigh 0), a NaN, coincident particles without softening.

Tolerance: every term is within a few units in the last place (2^-53), the
oracle adds up to N^2 / 2 terms one after another; 1e-11 of the sum of
magnitudes covers both for N <= 20000 many times over."""
import numpy as np
import pytest

import oracle
from gpu_helpers import gpu_view, say

import paper_2302_08251_amd as lm
from paper_2302_08251_amd import synth

pytestmark = pytest.mark.gpu

REC = ["f32"] * 7
EPS2 = float(np.float32(0.01))


def energies(planes, spec, eps2):
    v = gpu_view(REC, spec, len(planes[0]), oracle.store_planes(REC, spec, planes))
    e = lm.nbody_energy(v, eps2)
    pos = np.stack(planes[0:3], 1).astype(np.float64)
    vel = np.stack(planes[3:6], 1).astype(np.float64)
    m = planes[6].astype(np.float64)
    kin = 0.5 * float((m * (vel * vel).sum(1)).sum())
    return e, oracle.energy(pos, vel, m, eps2), kin


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 255, 256, 257, 511, 513, 769, 4097, 20000])
@pytest.mark.parametrize("spec", [{"kind": "aos"}, {"kind": "soa_mb"}], ids=["aos", "soa_mb"])
def test_energy_at_block_edges(n, spec):
    e, ref, kin = energies(synth.particles(n, n, dtype=np.float32), spec, EPS2)
    say("energy", n, spec["kind"], e, ref)
    assert abs(e - ref) <= 1e-11 * (kin + abs(ref - kin))


@pytest.mark.parametrize("n,at", [(300, 299), (600, 10), (1000, 256)])
def test_energy_of_values_outside_the_fast_form(n, at):
    planes = synth.particles(n, 5, dtype=np.float32)
    planes[1][at] = np.inf
    e, ref, kin = energies(planes, {"kind": "soa_mb"}, EPS2)
    say("inf position", n, at, e, ref)
    assert np.isfinite(ref) and abs(e - ref) <= 1e-11 * (kin + abs(ref - kin))
    planes[1][at] = np.nan
    assert np.isnan(energies(planes, {"kind": "soa_mb"}, EPS2)[0])
    planes = synth.particles(n, 6, dtype=np.float32)
    for p in planes[:3]:
        p[at] = p[(at + 1) % n]
    assert energies(planes, {"kind": "soa_mb"}, 0.0)[0] == -np.inf
