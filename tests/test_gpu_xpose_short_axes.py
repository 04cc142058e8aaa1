"""Row- to column-major copies whose fastest axes are short: tiles fitted to the
axes, of one column or (when they are small and many) of whole records, moved
by one wave or by four; both directions against the oracle's n-D copy, whole
blobs bit for bit, on both sides of each rule."""
import numpy as np
import pytest

import oracle
from gpu_helpers import assert_blobs_equal, bits_planes, download, say, upload

import paper_2302_08251_amd as lm

pytestmark = pytest.mark.gpu

AOS, SB, MB = {"kind": "aos"}, {"kind": "soa_sb"}, {"kind": "soa_mb"}
AO32, AO3 = {"kind": "aosoa", "lanes": 32}, {"kind": "aosoa", "lanes": 3}
BS = {"kind": "bytesplit", "inner": SB}
RECS = {"f32": ["f32"], "u8x3": ["u8"] * 3, "u16": ["u16"], "f32x3": ["f32"] * 3, "f64x5": ["f64"] * 5}


@pytest.mark.parametrize("ext", [(2, 5001, 2), (2, 300, 2), (16, 3, 301, 2), (3, 9001), (9001, 3), (1030, 2, 3), (5, 17, 1100),
                                 (17, 1100, 17), (4, 4, 4, 4, 4, 4), (31, 33, 65), (2, 2), (7, 9)])
@pytest.mark.parametrize("recname", sorted(RECS))
def test_short_axes(recname, ext):
    rec = RECS[recname]
    n = int(np.prod(ext))
    planes = bits_planes(n, rec, n)
    for k, (a, b) in enumerate(((AOS, MB), (SB, AOS), (SB, SB), (AOS, AOS), (AO32, MB), (MB, AO3), (BS, AOS), (MB, BS))):
        sc = bool((k + len(ext)) & 1) if n > 20000 else None
        for col in ((False, True) if sc is None else (sc,)):
            sa, sb = dict(a, col_major=col), dict(b, col_major=not col)
            say("short axes", recname, ext, sa, sb)
            src = oracle.store_planes(rec, sa, planes, fill=0x5A)
            exp = oracle.copy_nd(rec, sa, src, sb, list(ext), fill=0xA5)
            sv = lm.View(rec, sa, list(ext), blobs=upload(src))
            dv = lm.View(rec, sb, list(ext), fill=0xA5)
            lm.llama_copy(sv, dv)
            assert_blobs_equal(download(dv), exp, "%s -> %s %s" % (sa, sb, ext))
