"""Calls without a stream argument run on torch's current stream: the default one,
the stream of a context, and a stream under graph capture."""
import pytest

from gpu_helpers import say, torch

import paper_2302_08251_amd as lm

pytestmark = pytest.mark.gpu


def test_current_stream():
    t = torch()
    assert (lm._stream(None).value or 0) == t.cuda.current_stream().cuda_stream
    s = t.cuda.Stream()
    with t.cuda.stream(s):
        assert (lm._stream(None).value or 0) == s.cuda_stream != 0
    assert (lm._stream(s).value or 0) == s.cuda_stream


def test_capture():
    t = torch()
    a, b = lm.View(["f32"], {"kind": "aos"}, 1000, fill=3), lm.View(["f32"], {"kind": "soa_sb"}, 1000, fill=0)
    lm.llama_copy(a, b)
    t.cuda.synchronize()
    g = t.cuda.CUDAGraph()
    with t.cuda.graph(g):
        lm.llama_copy(a, b)
    for k in range(3):
        say("replay", k)
        b.blobs[0].zero_()
        a.blobs[0].fill_(k + 7)
        g.replay()
        t.cuda.synchronize()
        assert bool((b.blobs[0][:4000] == k + 7).all())
