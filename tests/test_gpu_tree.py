"""GPU parity of the tiled per-leaf and value-level copy with tiles of several
hundred records (record counts that give at least 512 such tiles), whole
blobs bit for bit against the oracle: partial last tiles, planes at odd
addresses, AoSoA blocks and record images inside a tile, codes across words,
byte columns, a SPLIT with a NULL part.  Smaller tiles: test_gpu_mixed.py,
test_gpu_generic.py."""
import pytest

import oracle
from gpu_helpers import assert_blobs_equal, bits_planes, download, gpu_view, say

import paper_2302_08251_amd as lm

pytestmark = pytest.mark.gpu

AOS, PACKED, SB, MB = {"kind": "aos"}, {"kind": "aos", "packed": True}, {"kind": "soa_sb"}, {"kind": "soa_mb"}
BS = {"kind": "bytesplit", "inner": {"kind": "soa_sb"}}
BSAO = {"kind": "bytesplit", "inner": {"kind": "aosoa", "lanes": 8}}


def ao(lanes):
    return {"kind": "aosoa", "lanes": lanes}


def ct(stored, inner):
    return {"kind": "changetype", "stored": stored, "inner": inner}


def bpi(bits):
    return {"kind": "bitpack_int", "bits": bits}


def bpf(E, M, **kw):
    return dict({"kind": "bitpack_float", "exp": E, "man": M}, **kw)


def split(at, a, b):
    return {"kind": "split", "at": at, "parts": [a, b]}


EVENT = ["u8", "f64", "i16", "f32"]
I3 = ["i32", "u16", "i64"]
F3 = ["f32", "f64", "f32"]
CASES = [
    (EVENT, AOS, MB), (EVENT, SB, AOS), (EVENT, PACKED, ao(32)), (EVENT, ao(24), PACKED), (EVENT, SB, BS),
    (EVENT, BSAO, AOS), (EVENT, MB, split(2, ao(32), PACKED)), (EVENT, split(1, SB, ao(3)), PACKED),
    (EVENT, split(3, PACKED, {"kind": "null"}), MB),
    (I3, MB, ct(["i16", "u8", "i32"], SB)), (I3, ct(["i16", "u32", "i8"], AOS), bpi(12)), (I3, bpi(9), bpi(16)),
    (I3, bpi(11), ct(["i64", "u16", "i32"], ao(40))), (I3[2:], AOS, bpi(41)), (I3[2:], bpi(63), SB),
    (F3, bpf(8, 15), bpf(5, 10)), (F3, bpf(5, 9), bpf(8, 12, round="rne")), (F3, ct(["f16", "f32", "f64"], SB), bpf(6, 13)),
    (["u8", "i16", "f32", "u8", "f64", "u16"], MB, AOS), (["u16", "u8", "u16", "u8", "i32"], split(3, AOS, MB), split(4, AOS, SB)),
    (["f16", "bf16"], bpf(4, 7), ao(16)), (F3, bpf(8, 7), ct(["bf16", "f16", "f32"], AOS)),
]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("n", [1000003, 1000064])
def test_tiles_of_many_records(case, n):
    rec, a, b = CASES[case]
    planes = bits_planes(n, rec, seed=case)
    say("tree", rec, a, b, n)
    src = oracle.store_planes(rec, a, planes, fill=0x5A)
    sv, dv = gpu_view(rec, a, n, src), gpu_view(rec, b, n, fill=0xA5)
    lm.llama_copy(sv, dv)
    assert_blobs_equal(download(dv), oracle.copy(rec, a, src, b, n, fill=0xA5), "%s -> %s" % (a, b))
