"""Packs and unpacks at the edges of their plan's rules: into AoS through the record
image (field counts that are no multiple of four, up to the 256-record tile) and
gathered, AoSoA blocks by quads and gathered, AoS records of a multiple of 32
bytes into the word image, one plane whose length is no multiple of four, few and
many tiles; whole blobs bit for bit."""
import pytest

import oracle
from gpu_helpers import assert_blobs_equal, bits_planes, download, gpu_view, say

import paper_2302_08251_amd as lm

pytestmark = pytest.mark.gpu

AOS, SB, MB = {"kind": "aos"}, {"kind": "soa_sb"}, {"kind": "soa_mb"}
AO32, AO6 = {"kind": "aosoa", "lanes": 32}, {"kind": "aosoa", "lanes": 6}


def run(rec, a, b, n):
    say("rules", len(rec), rec[0], a, b, n)
    src = oracle.store_planes(rec, a, bits_planes(n, rec, seed=n + len(rec)), fill=0x5A)
    sv, dv = gpu_view(rec, a, n, src), gpu_view(rec, b, n, fill=0xA5)
    lm.llama_copy(sv, dv)
    assert_blobs_equal(download(dv), oracle.copy(rec, a, src, b, n, fill=0xA5), "%s -> %s" % (a, b))


@pytest.mark.parametrize("n", [5, 255, 1027, 30011])
@pytest.mark.parametrize("nf", [1, 2, 3, 4, 6, 7, 8, 15, 16, 17, 40])
def test_field_counts(nf, n):
    ints, floats = {"kind": "bitpack_int", "bits": 29}, {"kind": "bitpack_float", "exp": 8, "man": 15}
    for lay in (AOS, AO32, AO6, SB, MB):
        run(["i32"] * nf, {"kind": "bitpack_int", "bits": 5}, lay, n)
        run(["i32"] * nf, lay, ints, n)
        run(["f32"] * nf, floats, lay, n)
        run(["f32"] * nf, lay, floats, n)


@pytest.mark.parametrize("nf,n", [(1, 4200003), (2, 2100003), (4, 1048575), (4, 1048577), (7, 600001)])
def test_few_and_many_tiles(nf, n):
    for lay in (AOS, SB, MB):
        run(["i32"] * nf, lay, {"kind": "bitpack_int", "bits": 16}, n)
        run(["i32"] * nf, lay, {"kind": "bitpack_int", "bits": 7}, n)
        run(["i32"] * nf, {"kind": "bitpack_int", "bits": 24}, lay, n)
