"""Per-leaf and value-level copies through AoSoA blocks of one record, plain and
under Bytesplit, whose byte columns then lie a whole record apart: as source,
as destination, under ChangeType, against codes and as a part of a SPLIT, at
record counts below, at and above a tile, whole blobs bit for bit."""
import pytest

import oracle
from gpu_helpers import assert_blobs_equal, bits_planes, download, gpu_view, say

import paper_2302_08251_amd as lm

pytestmark = pytest.mark.gpu

AOS, PACKED, SB, MB = {"kind": "aos"}, {"kind": "aos", "packed": True}, {"kind": "soa_sb"}, {"kind": "soa_mb"}
AO1 = {"kind": "aosoa", "lanes": 1}
BS, BS1 = {"kind": "bytesplit", "inner": SB}, {"kind": "bytesplit", "inner": AO1}


def ct(stored, inner):
    return {"kind": "changetype", "stored": stored, "inner": inner}


def split(at, a, b):
    return {"kind": "split", "at": at, "parts": [a, b]}


EVENT = ["u8", "f64", "i16", "f32"]
I3, S3 = ["i32"] * 3, ["i16"] * 3
F7 = ["f32"] * 7
CASES = [
    (EVENT, BS1, MB), (EVENT, MB, BS1), (EVENT, BS1, BS1), (EVENT, BS1, BS), (EVENT, BS, BS1),
    (EVENT, AO1, MB), (EVENT, SB, AO1), (EVENT, AO1, AOS), (EVENT, BS1, AO1), (EVENT, PACKED, BS1),
    (I3, ct(S3, BS1), AOS), (I3, AOS, ct(S3, BS1)), (I3, ct(S3, BS1), {"kind": "bitpack_int", "bits": 12}),
    (I3, {"kind": "bitpack_int", "bits": 12}, ct(S3, BS1)), (I3, ct(S3, AO1), ct(S3, BS1)),
    (F7, split(3, BS1, SB), AOS), (F7, AOS, split(3, SB, BS1)), (F7, split(2, BS1, AO1), split(5, MB, BS1)),
    (EVENT, split(1, AOS, BS1), PACKED), (EVENT, split(3, BS1, {"kind": "null"}), MB),
]


@pytest.mark.parametrize("n", [1, 5, 256, 4099, 300007])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_one_lane(case, n):
    rec, a, b = CASES[case]
    planes = bits_planes(n, rec, seed=case + n)
    say("one lane", rec, a, b, n)
    src = oracle.store_planes(rec, a, planes, fill=0x5A)
    sv, dv = gpu_view(rec, a, n, src), gpu_view(rec, b, n, fill=0xA5)
    lm.llama_copy(sv, dv)
    assert_blobs_equal(download(dv), oracle.copy(rec, a, src, b, n, fill=0xA5), "%s -> %s" % (a, b))
