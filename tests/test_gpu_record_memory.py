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

    g, o = pair(lda_mod, oracle_mod, doff, words, 50, 1564, dev_alloc=alloc, dev_free=free,
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


@pytest.mark.parametrize("opt", [{}, {"dense_rows": 12, "dense_alias_min_count": 1 << 20},
                                 {"record_bucket_tokens": 512}, {"stream_block_tokens": 3000}])
def test_a_failed_init_gives_back_idle_memory(lda_mod, opt):
    """lda_init behind other work on its stream, with an allocator that fails at the first, the
    second, ... request: every block comes back, and only when the stream is idle."""
    rng = np.random.default_rng(2)
    doff = np.arange(0, 10_001, 100, dtype=np.int64)
    words = rng.integers(0, 30, 10_000).astype(np.int32)
    stream = torch.cuda.Stream()
    busy = torch.zeros(1 << 26, device="cuda")
    torch.cuda.synchronize()
    live, idle, left = {}, [], [0]

    def alloc(nbytes):
        if left[0] == 0:
            return 0
        left[0] -= 1
        t = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        live[t.data_ptr()] = t
        return t.data_ptr()

    def free(p):
        idle.append(stream.query())
        assert p in live
        back.append(live.pop(p))  # held until the next attempt

    for budget in range(1, 200):
        left[0], back = budget, []
        with torch.cuda.stream(stream):
            for _ in range(10):
                busy.add_(1.0)
        try:
            g = lda_mod.Lda(doff, words, 30, 20, 0.1, 0.01, dev_alloc=alloc, dev_free=free,
                            stream=stream.cuda_stream, **opt)
        except lda_mod.LdaError as e:
            assert e.code == lda_mod.LDA_ERR_OOM
            assert not live and len(back) == budget
        else:
            g.close()
            break
        torch.cuda.synchronize()
    assert 20 < budget < 199 and not live and all(idle)


# bytes per token that the allocator grants: two steps use 4 for the word-major records and 16 for
# the others, four steps 8 and 32; 0: not even what was given back
@pytest.mark.parametrize("grant", [0, 6, 10, 20])
def test_out_of_memory_leaves_a_usable_context(lda_mod, oracle_mod, grant):
    doff, words = make(50, 7, docs=300)
    N = int(doff[-1])
    limit, live = [1 << 60], {}

    def alloc(nbytes):
        if nbytes > limit[0]:
            return 0
        t = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        live[t.data_ptr()] = t
        return t.data_ptr()

    g, o = pair(lda_mod, oracle_mod, doff, words, 50, 64, dev_alloc=alloc, dev_free=lambda p: live.pop(p))
    sweep_both(g, o, 2)
    g.build_alias()
    limit[0] = grant * N
    with pytest.raises(lda_mod.LdaError) as e:
        g.sweep(4)
    assert e.value.code == lda_mod.LDA_ERR_OOM
    if grant:  # the word-major records are there again
        g.rebuild_counts()
        assert np.array_equal(g.get_nk(), o.get_nk())
    else:
        with pytest.raises(lda_mod.LdaError) as e:
            g.rebuild_counts()
        assert e.value.code == lda_mod.LDA_ERR_OOM
    if grant in (6, 20):
        sweep_both(g, o, 2)
    limit[0] = 1 << 60
    for m in (2, 4, 1):
        sweep_both(g, o, m)
    g.close(); o.close()
    assert not live


def test_records_that_grow_in_a_graph(lda_mod, oracle_mod):
    """While its stream is captured a sweep may take larger records from the caller's allocator; the
    old ones, which earlier work may still use, stay until lda_destroy."""
    doff, words = make(50, 11, docs=300)
    pool = torch.empty(1 << 26, dtype=torch.uint8, device="cuda")  # handed out piece by piece
    used, live, freed = [0], set(), []

    def alloc(nbytes):
        at = used[0]
        used[0] += (nbytes + 255) // 256 * 256
        assert used[0] <= len(pool)
        live.add(pool.data_ptr() + at)
        return pool.data_ptr() + at

    def free(p):
        live.remove(p)
        freed.append(p)

    stream = torch.cuda.Stream()
    g, o = pair(lda_mod, oracle_mod, doff, words, 50, 64, dev_alloc=alloc, dev_free=free,
                stream=stream.cuda_stream)
    sweep_both(g, o, 2)
    g.build_alias(); o.build_alias()
    g.sync()
    before, taken = len(freed), used[0]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        g.sweep(4)
    assert len(freed) == before and used[0] > taken
    o.sweep(4)
    for i in range(3):
        with torch.cuda.stream(stream):
            graph.replay()
        assert np.array_equal(g.get_z(), o.get_z()), i
        torch.cuda.synchronize()
    g.rebuild_counts(); o.rebuild_counts()
    assert np.array_equal(g.get_nk(), o.get_nk())
    for m in (4, 2, 3):
        sweep_both(g, o, m)
    assert len(freed) == before
    g.close(); o.close()
    assert not live
