"""Chains of 5 to 8 steps: in two passes where that gains and their records can be had, otherwise
(and beyond 8 steps) in one; against the oracle, bit for bit, in every store and in turn with other
chains.  The corpora of make() have long documents, so they take two passes from K * steps = 7500 on
(1500 with words of the mixture)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lda_mod():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_1412_1576_amd import lda
    lda.load_library()
    return lda


def make(V, seed, docs=150):
    rng = np.random.default_rng(seed)
    # around a tile, longer than one (a document of its own workgroup), empty ones
    lens = [0, 1024, 3, 1025, 1, 0, 1023, 2500, 512, 63] + list(rng.integers(0, 130, docs)) + [0]
    doff = np.zeros(len(lens) + 1, np.int64)
    doff[1:] = np.cumsum(lens)
    p = 1.0 / np.arange(1, V + 1)
    return doff, rng.choice(V, int(doff[-1]), p=p / p.sum()).astype(np.int32)


def pair(lda_mod, oracle_mod, doff, words, V, K, **opt):
    g = lda_mod.Lda(doff, words, V, K, 0.1, 0.01, seed=5, **opt)
    o = oracle_mod.Oracle(doff, words, V, K, 0.1, 0.01, seed=5,
                          dense_alias_min_count=opt.get("dense_alias_min_count", 0))
    return g, o


def sweep_both(g, o, m):
    g.build_alias(); o.build_alias()
    g.sweep(m); o.sweep(m)
    g.rebuild_counts(); o.rebuild_counts()
    assert np.array_equal(g.get_z(), o.get_z()), m
    assert np.array_equal(g.get_nk(), o.get_nk()), m


# rows staged in LDS and gathered (dense), staged and gathered mixture rows, rows beyond LDS, no
# dense rows, n_k gathered (K > 16384), topics of more than 16 bits
@pytest.mark.parametrize("V,K,dense_rows", [(90, 33, 0), (90, 1510, 0), (300, 1000, 300), (40, 13000, 25),
                                            (90, 17001, -1), (40, 66000, 3)])
@pytest.mark.parametrize("m", [5, 6, 7, 8])
def test_steps_and_stores(lda_mod, oracle_mod, V, K, dense_rows, m):
    doff, words = make(V, 10 * m + V)
    cnt = np.bincount(words, minlength=V)
    opt = {}
    if dense_rows:
        tail = cnt[max(dense_rows, 0):]
        opt = {"dense_rows": dense_rows, "dense_alias_min_count": int(tail.max()) + 1 if len(tail) else 400}
    g, o = pair(lda_mod, oracle_mod, doff, words, V, K, **opt)
    for steps in (m, m, 2, m, 9, m):
        sweep_both(g, o, steps)
    g.close(); o.close()


def test_record_buckets(lda_mod, oracle_mod):
    doff, words = make(50, 3)
    g, o = pair(lda_mod, oracle_mod, doff, words, 50, 1570, record_bucket_tokens=512)
    for steps in (8, 7, 8, 5, 6):
        sweep_both(g, o, steps)
    g.close(); o.close()


def test_no_room_for_the_records(lda_mod, oracle_mod):
    """An allocator that refuses the records of a long chain, the first or the second of them: the
    sweep runs without them, and what was there before stays usable."""
    doff, words = make(50, 4, docs=600)
    left, live = [1 << 60], set()

    def alloc(nbytes):
        if nbytes > left[0]:
            return 0
        p = torch.cuda.caching_allocator_alloc(nbytes, 0)
        live.add(p)
        return p

    def free(p):
        live.remove(p)
        torch.cuda.synchronize()
        torch.cuda.caching_allocator_delete(p)

    N = int(doff[-1])
    for limit in (N, 20 * N, 1 << 60):
        left[0] = 1 << 60
        g, o = pair(lda_mod, oracle_mod, doff, words, 50, 1564, dev_alloc=alloc, dev_free=free)
        sweep_both(g, o, 2)
        left[0] = limit
        n = len(live)
        for steps in (8, 2, 6):
            sweep_both(g, o, steps)
        assert len(live) == n
        g.close(); o.close()
        assert not live


def test_a_refusal_is_remembered(lda_mod, oracle_mod):
    """Refused records are no error, are asked for once, and again only if a chain needs less."""
    doff, words = make(50, 8, docs=600)
    N = int(doff[-1])
    left, live, asked = [1 << 60], {}, []

    def alloc(nbytes):
        asked.append(nbytes)
        if nbytes > left[0]:
            return 0
        left[0] -= nbytes
        t = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        live[t.data_ptr()] = t
        return t.data_ptr()

    def free(p):
        left[0] += len(live.pop(p))

    g, o = pair(lda_mod, oracle_mod, doff, words, 50, 1564, dev_alloc=alloc, dev_free=free)
    sweep_both(g, o, 2)
    left[0] = 75 * N  # 8 steps take 64 and 16 bytes per token, 5 steps 64 and 8
    seen = []
    for steps in (8, 8, 7, 2, 8, 5, 6, 8, 8):
        del asked[:]
        sweep_both(g, o, steps)
        seen.append([n // N for n in asked])
        assert not lda_mod.load_library().lda_last_error(g._h), steps
    assert seen == [[64, 16], [], [64, 8], [], [16], [], [], [], []], seen
    g.close(); o.close()
    assert not live


def test_first_long_chain_in_a_graph(lda_mod, oracle_mod):
    """While its stream is captured a sweep allocates nothing: it runs without records, and the
    graph gives the oracle's assignment at every replay.  The next sweep asks for the records."""
    doff, words = make(50, 9, docs=600)
    N = int(doff[-1])
    live, asked = {}, []

    def alloc(nbytes):
        asked.append(nbytes // N)
        t = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        live[t.data_ptr()] = t
        return t.data_ptr()

    stream = torch.cuda.Stream()
    g, o = pair(lda_mod, oracle_mod, doff, words, 50, 1564, dev_alloc=alloc, dev_free=lambda p: live.pop(p),
                stream=stream.cuda_stream)
    sweep_both(g, o, 2)
    g.build_alias(); o.build_alias()
    g.sync()
    other = torch.ones(1 << 20, device="cuda")
    graph = torch.cuda.CUDAGraph()
    del asked[:]
    with torch.cuda.graph(graph, stream=stream):
        g.sweep(8)
    assert not asked
    o.sweep(8)
    for i in range(3):
        with torch.cuda.stream(stream):
            graph.replay()
            other.mul_(2.0)
        assert np.array_equal(g.get_z(), o.get_z()), i
        torch.cuda.synchronize()
    g.rebuild_counts(); o.rebuild_counts()
    assert np.array_equal(g.get_nk(), o.get_nk())
    assert not asked
    sweep_both(g, o, 8)
    assert asked == [64, 16]
    sweep_both(g, o, 2)
    g.close(); o.close()


# corpora on both sides of the rule: tokens, length of most documents, tokens of one long document,
# words, K, dense_alias_min_count, steps, whether the records are asked for
@pytest.mark.parametrize("N,L,long,V,K,below,m,two", [
    (100_000, 90, 0, 50, 64, 0, 5, False), (100_000, 90, 0, 900, 2000, 0, 8, False),
    (100_000, 90, 0, 900, 2000, 2000, 8, False),
    (100_000, 90, 4000, 50, 937, 0, 8, False), (100_000, 90, 4000, 50, 938, 0, 8, True),
    (100_000, 90, 4000, 900, 299, 900, 5, False), (100_000, 90, 4000, 900, 300, 900, 5, True),
    (100_000, 90, 3000, 900, 300, 900, 5, False), (1_200_000, 90, 40_000, 50, 2000, 0, 8, False),
    (1_200_000, 90, 40_000, 9000, 600, 600, 5, True), (1_200_000, 90, 0, 9000, 600, 600, 5, False),
    (3_000_000, 90, 0, 9000, 600, 600, 5, True), (3_000_000, 90, 0, 9000, 599, 599, 5, False),
    (3_000_000, 90, 0, 9000, 600, 2, 5, False), (3_000_000, 90, 0, 9000, 600, 0, 8, False)])
def test_which_form(lda_mod, N, L, long, V, K, below, m, two):
    rng = np.random.default_rng(N + K)
    words = (V * rng.random(N) ** 4).astype(np.int32)
    doff = np.append(np.arange(0, N - long, L), [N - long, N] if long else [N]).astype(np.int64)
    live, asked = {}, []

    def alloc(nbytes):
        asked.append(nbytes)
        t = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        live[t.data_ptr()] = t
        return t.data_ptr()

    g = lda_mod.Lda(doff, words, V, K, 0.1, 0.01, seed=1, dev_alloc=alloc, dev_free=lambda p: live.pop(p),
                    dense_alias_min_count=below)
    g.build_alias()
    del asked[:]
    g.sweep(m)
    assert (64 * N in asked) == two, asked
    g.rebuild_counts()
    assert np.array_equal(g.get_nk(), np.bincount(g.get_z(), minlength=K))
    g.close()
