"""The records of the sweep's two passes, which grow with the longest chain asked for: what happens
to the memory they had before, with a caller's allocator."""
import numpy as np
import pytest
import torch

from test_gpu_long_chains import lda_mod, make, pair, sweep_both  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("steps", [(2, 4), (2, 8), (4, 8), (1, 5)])
def test_given_back_when_no_longer_used(lda_mod, oracle_mod, steps):
    """A block goes back to the caller, who may hand it on at once, when the stream is idle."""
    doff, words = make(50, 6, docs=600)
    stream = torch.cuda.Stream()
    live, idle = {}, []

    def alloc(nbytes):
        t = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        live[t.data_ptr()] = t  # held to the end of the test: nothing is handed on here
        return t.data_ptr()

    def free(p):
        idle.append(stream.query())

    g, o = pair(lda_mod, oracle_mod, doff, words, 50, 64, dev_alloc=alloc, dev_free=free,
                stream=stream.cuda_stream)
    busy = torch.zeros(1 << 28, device="cuda")
    torch.cuda.synchronize()
    for m in steps:
        g.build_alias(); o.build_alias()
        with torch.cuda.stream(stream):
            for _ in range(40):
                busy.add_(1.0)
        del idle[:]
        g.sweep(m); o.sweep(m)
        given_back = list(idle)
        g.rebuild_counts(); o.rebuild_counts()
        assert np.array_equal(g.get_z(), o.get_z()), m
    assert given_back and all(given_back), (steps, given_back)
    g.close(); o.close()
