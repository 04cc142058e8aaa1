"""The n-body step with a particle of infinite mass: every other particle's
acceleration is an infinity towards it, as the plain float32 sum gives it
(one pair is infinite, every other is finite), whichever j tile and slice the
particle lies in; the particle's own is 0 * inf, a NaN.  Exact: no tolerance."""
import numpy as np
import pytest

import oracle
from gpu_helpers import download, gpu_view, say

import paper_2302_08251_amd as lm
from paper_2302_08251_amd import synth

pytestmark = pytest.mark.gpu

REC = ["f32"] * 7
EPS2, DT = 0.01, 1e-4


@pytest.mark.parametrize("n", [300, 512, 1000, 4096, 20000])
@pytest.mark.parametrize("where", ["first", "middle", "last"])
def test_infinite_mass(n, where):
    at = {"first": 0, "middle": n // 2, "last": n - 1}[where]
    planes = synth.particles(n, 7, dtype=np.float32)
    planes[6][at] = np.inf
    say("infinite mass", n, at)
    v = gpu_view(REC, {"kind": "soa_mb"}, n, oracle.store_planes(REC, {"kind": "soa_mb"}, planes))
    lm.nbody_step(v, 1, DT, EPS2)
    got = oracle.load_planes(REC, {"kind": "soa_mb"}, download(v), n)
    others = np.arange(n) != at
    for c in range(3):
        d = planes[c][at] - planes[c]
        want = np.where(d > 0, np.float32(np.inf), np.float32(-np.inf))
        check = others & (d != 0)
        assert check.sum() > n // 2
        assert np.array_equal(got[3 + c][check], want[check])
        assert np.array_equal(got[c][check], want[check])
        assert np.isnan(got[3 + c][at])
