"""GPU parity of the line-owner writes (single-blob planes off the 128-byte line
grid) around the edges of their tiles (384 and 768 records and their halos), for
leaves of 2, 4 and 8 bytes, whole blobs bit for bit against the oracle."""
import pytest

import oracle
from gpu_helpers import CFG2, assert_blobs_equal, bits_planes, download, gpu_view, say

import paper_2302_08251_amd as lm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [5, 127, 383, 385, 415, 767, 769, 897, 1537, 50001])
@pytest.mark.parametrize("rec", [["f64"] * 7, ["f32"] * 3, ["u16"] * 5], ids=lambda r: "%sx%d" % (r[0], len(r)))
def test_line_tiles(rec, n):
    planes = bits_planes(n, rec, seed=n)
    for a in CFG2:
        src = oracle.store_planes(rec, CFG2[a], planes, fill=0x5A)
        for b in ("soa_sb", "bytesplit"):
            say("line", rec, a, b, n)
            sv, dv = gpu_view(rec, CFG2[a], n, src), gpu_view(rec, CFG2[b], n, fill=0xA5)
            lm.llama_copy(sv, dv)
            assert_blobs_equal(download(dv), oracle.copy(rec, CFG2[a], src, CFG2[b], n, fill=0xA5), "%s -> %s n=%d" % (a, b, n))
