"""Row- to column-major copies at the edges of the transpose's tiles (runs of 16
to 128 records, one column per tile or whole records), in both directions and
against the oracle's n-D copy, whole blobs bit for bit: extents one off the
edges, many tiles, records of one column, records too wide for a full tile."""
import numpy as np
import pytest

import oracle
from gpu_helpers import assert_blobs_equal, bits_planes, download, say, upload

import paper_2302_08251_amd as lm

pytestmark = pytest.mark.gpu

AOS, SB, MB = {"kind": "aos"}, {"kind": "soa_sb"}, {"kind": "soa_mb"}
AO24 = {"kind": "aosoa", "lanes": 24}
BS = {"kind": "bytesplit", "inner": {"kind": "soa_sb"}}
RECS = {"f32": ["f32"], "f32x3": ["f32"] * 3, "u16x3": ["u16"] * 3, "u8x2": ["u8"] * 2, "f64x7": ["f64"] * 7,
        "f64x40": ["f64"] * 40}


@pytest.mark.parametrize("ext", [(63, 65), (129, 31), (1, 700), (515, 513), (33, 7, 129), (200, 2, 3, 65)])
@pytest.mark.parametrize("recname", sorted(RECS))
def test_tile_edges(recname, ext):
    rec = RECS[recname]
    if len(rec) >= 7 and np.prod(ext) > 50000:
        ext = (257, 129)
    n = int(np.prod(ext))
    planes = bits_planes(n, rec, n)
    for k, (a, b) in enumerate(((AOS, MB), (SB, AOS), (SB, SB), (AOS, AOS), (AO24, MB), (MB, AO24)) + (((BS, AOS), (MB, BS)) if len(rec) <= 7 else ())):
        for sc in ((False, True) if n < 50000 else (bool(k & 1),)):
            sa, sb = dict(a, col_major=sc), dict(b, col_major=not sc)
            say("xpose", recname, ext, sa, sb)
            src = oracle.store_planes(rec, sa, planes, fill=0x5A)
            exp = oracle.copy_nd(rec, sa, src, sb, list(ext), fill=0xA5)
            sv = lm.View(rec, sa, list(ext), blobs=upload(src))
            dv = lm.View(rec, sb, list(ext), fill=0xA5)
            lm.llama_copy(sv, dv)
            assert_blobs_equal(download(dv), exp, "%s -> %s %s" % (sa, sb, ext))
