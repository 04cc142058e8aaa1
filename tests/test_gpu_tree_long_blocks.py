"""Per-leaf and value-level copies through AoSoA blocks whose tiles hold more than
1024 records (9, 17 and 100 lanes), that fit no tile (33 and 250 lanes), on both
sides of the record counts from which the tiled form takes them, whole blobs bit
for bit."""
import pytest

import oracle
from gpu_helpers import assert_blobs_equal, bits_planes, download, gpu_view, say

import paper_2302_08251_amd as lm

pytestmark = pytest.mark.gpu

MB, BS = {"kind": "soa_mb"}, {"kind": "bytesplit", "inner": {"kind": "soa_sb"}}
EVENT = ["u8", "f64", "i16", "f32"]


def forms(lanes):
    ao = {"kind": "aosoa", "lanes": lanes}
    return [(EVENT, ao, MB), (EVENT, BS, ao), (["i32"] * 3, {"kind": "changetype", "stored": ["i16"] * 3, "inner": ao},
                                              {"kind": "bitpack_int", "bits": 12})]


@pytest.mark.parametrize("lanes,ns", [(9, (512, 513, 293761, 294913)), (17, (500, 4097, 557100)), (100, (512, 9910, 819201)),
                                      (33, (100, 9000)), (250, (100, 9000))])
@pytest.mark.parametrize("form", range(3))
def test_long_blocks(lanes, ns, form):
    rec, a, b = forms(lanes)[form]
    for n in ns:
        say("long blocks", lanes, n, a, b)
        src = oracle.store_planes(rec, a, bits_planes(n, rec, seed=n + form), fill=0x5A)
        sv, dv = gpu_view(rec, a, n, src), gpu_view(rec, b, n, fill=0xA5)
        lm.llama_copy(sv, dv)
        assert_blobs_equal(download(dv), oracle.copy(rec, a, src, b, n, fill=0xA5), "%s -> %s n=%d" % (a, b, n))
