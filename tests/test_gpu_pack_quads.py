"""GPU parity of packs and unpacks that move four records of a field per lane,
whole blobs bit for bit against the oracle: record-major, blocked and planar
sides on and off the 16-byte grid, code widths with and without whole words
per quad, partial quads, groups and tiles, and explicit tiles whose record image
would not fit in LDS."""
import pytest

import oracle
from gpu_helpers import F32x7, assert_blobs_equal, bits_planes, download, gpu_view, say

import paper_2302_08251_amd as lm

pytestmark = pytest.mark.gpu

LAYOUTS = [{"kind": "aos"}, {"kind": "soa_sb"}, {"kind": "soa_mb"}, {"kind": "aosoa", "lanes": 32},
           {"kind": "aosoa", "lanes": 4}, {"kind": "aosoa", "lanes": 6}]


def bpf(E, M, **kw):
    return dict({"kind": "bitpack_float", "exp": E, "man": M}, **kw)


def bpi(bits):
    return {"kind": "bitpack_int", "bits": bits}


CODES = [(F32x7, bpf(8, 15)), (F32x7, bpf(5, 10)), (F32x7, bpf(8, 23)), (F32x7, bpf(4, 3)), (F32x7, bpf(6, 13, round="rne")),
         (["i32"] * 3, bpi(24)), (["u32"] * 3, bpi(5)), (["i32"] * 3, bpi(13)), (["i32"] * 3, bpi(31)), (["u32"], bpi(32))]


def both_ways(rec, spec, layout, n, tile=0):
    planes = bits_planes(n, rec, seed=n + spec.get("bits", spec.get("man", 0)))
    src = oracle.store_planes(rec, layout, planes, fill=0x5A)
    code = oracle.copy(rec, layout, src, spec, n, fill=0xA5)
    back = oracle.copy(rec, spec, code, layout, n, fill=0xA5)
    sv, cv, bv = gpu_view(rec, layout, n, src), gpu_view(rec, spec, n, fill=0xA5), gpu_view(rec, layout, n, fill=0xA5)
    lm.llama_copy_ex(sv, cv, tile_records=tile)
    assert_blobs_equal(download(cv), code, "pack %s %s n=%d tile=%d" % (layout, spec, n, tile))
    lm.llama_copy_ex(cv, bv, tile_records=tile)
    assert_blobs_equal(download(bv), back, "unpack %s %s n=%d tile=%d" % (layout, spec, n, tile))


@pytest.mark.parametrize("n", [1, 3, 4, 255, 257, 1030, 50001])
@pytest.mark.parametrize("code", range(len(CODES)))
def test_quads(code, n):
    rec, spec = CODES[code]
    for layout in LAYOUTS:
        say("quads", rec, spec, layout, n)
        both_ways(rec, spec, layout, n)


@pytest.mark.parametrize("tile", [384, 1152, 1536])
def test_explicit_tiles(tile):
    """1152 records of 7 x f32 and their 24-bit codes leave room for the record
    image, 1536 do not."""
    for layout in LAYOUTS[:4]:
        say("quads tile", layout, tile)
        both_ways(F32x7, bpf(8, 15), layout, 5003, tile)
