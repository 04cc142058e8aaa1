"""Copies whose tiles outnumber the workgroups of one launch (a launch takes fewer
than 2^32 threads, 2^24 workgroups of 256): a transpose of short outer axes, whose
middle axis makes one tile each, and codes of 1 bit to codes of 2 bits, whose
tiles of 4096 records are full at 2^36 records (8 GiB to 16 GiB)."""
import numpy as np
import pytest

from gpu_helpers import say, torch

import paper_2302_08251_amd as lm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("middle", [(1 << 24) - 1, 1 << 24, (1 << 24) + 77])
def test_transpose_of_many_tiles(middle):
    t = torch()
    ext = [2, middle, 2]
    say("transpose", ext)
    src = t.randint(0, 256, (2, middle, 2), dtype=t.uint8, device="cuda")
    sv = lm.View(["u8"], {"kind": "aos"}, ext, blobs=[src.reshape(-1)])
    dv = lm.View(["u8"], {"kind": "soa_mb", "col_major": True}, ext, fill=0)
    lm.llama_copy(sv, dv)
    got = dv.blobs[0][: 4 * middle].reshape(2, middle, 2)
    assert t.equal(got, src.permute(2, 1, 0))


def test_codes_of_many_tiles():
    t = torch()
    n = (1 << 36) + 4096 * 3 + 5
    sv = lm.View(["u8"], {"kind": "bitpack_int", "bits": 1}, [n], index_type="i64")
    dv = lm.View(["u8"], {"kind": "bitpack_int", "bits": 2}, [n], index_type="i64", fill=0xA5)
    say("codes", n, sv.sizes, dv.sizes)
    src = sv.blobs[0]
    src[src.numel() - src.numel() % 8:].zero_()
    whole = src[: src.numel() // 8 * 8].view(t.int64)
    whole.random_()
    src[n // 8 + 1: sv.sizes[0]].zero_()
    src[n // 8] &= (1 << n % 8) - 1  # the bits past the last code are 0
    lm.llama_copy(sv, dv)
    bit = t.arange(8, device="cuda", dtype=t.int32)
    for b0 in (0, 1 << 20, (1 << 33) - 4096, n // 8 - 70000):
        part = src[b0: min(b0 + (1 << 17), n // 8)].to(t.int32)
        codes = (part[:, None] >> bit) & 1
        want = (codes.reshape(-1, 4) << (2 * bit[:4])).sum(1).to(t.uint8)
        assert t.equal(dv.blobs[0][2 * b0: 2 * b0 + want.numel()], want)
    last = [int(src[n // 8]) >> k & 1 for k in range(n % 8)]
    tail = dv.blobs[0][2 * (n // 8): dv.sizes[0]].cpu().numpy().astype(np.int64)
    assert [int(tail[k // 4]) >> 2 * (k % 4) & 3 for k in range(n % 8)] == last
