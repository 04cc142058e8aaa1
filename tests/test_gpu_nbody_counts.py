"""Access counters of the n-body consumer over several j slices and i blocks, with
short last j tiles and waves: FieldAccessCount, and Heatmaps of counters that
neighbouring elements share, that hold one element each and that one element
spans, against the oracle's n-body through the same mapping, bit for bit."""
import numpy as np
import pytest

import oracle
from gpu_helpers import assert_blobs_equal, download, gpu_view, say

import paper_2302_08251_amd as lm
from paper_2302_08251_amd import synth

pytestmark = pytest.mark.gpu

REC = ["f32"] * 7


def heat(inner, g):
    return {"kind": "heatmap", "granularity": g, "inner": inner}


@pytest.mark.parametrize("n", [1, 63, 65, 700, 2500, 5003])
@pytest.mark.parametrize("spec", [{"kind": "field_access_count", "inner": {"kind": "aos"}}, heat({"kind": "soa_mb"}, 4),
                                  heat({"kind": "soa_sb"}, 1), heat({"kind": "aos"}, 64), heat({"kind": "aosoa", "lanes": 3}, 2),
                                  heat({"kind": "soa_mb"}, 1 << 20)],
                         ids=["fac", "heat4_mb", "heat1_sb", "heat64_aos", "heat2_aosoa3", "heat1M_mb"])
def test_counts_over_slices(spec, n):
    planes = [p.astype(np.float32) for p in synth.particles(n, 4)]
    host = oracle.store_planes(REC, spec, planes, fill=0)
    nin = oracle.blob_count(REC, spec["inner"])
    for b in host[nin:]:
        b[:] = 0
    say("counts", spec, n)
    v = gpu_view(REC, spec, n, host)
    lm.nbody_step(v, 1, 1e-4, 0.01)
    got = download(v)
    oracle.nbody_view(REC, spec, host, n, 1, 1e-4, 0.01, tile=256)
    assert_blobs_equal(got[nin:], host[nin:], "counters")
    v.close()
