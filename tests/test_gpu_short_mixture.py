"""Mixture words with few tokens, which the word pass serves from their lists in LDS: the ends of the form
(1024 tokens and one more, 512 words to a piece, words without tokens, K / 8 tokens), on dense rows,
on rows that only exist as lists and on hash rows, with every chain shape, against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lda_mod():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_1412_1576_amd import lda
    lda.load_library()
    return lda


def corpus_of(counts, seed):
    words = np.repeat(np.arange(len(counts), dtype=np.int32), counts)
    np.random.default_rng(seed).shuffle(words)
    return np.append(np.arange(0, len(words), 90), len(words)).astype(np.int64), words


@pytest.mark.parametrize("K", [100, 1000, 8200, 16385, 36864, 36865, 100001, 1000003])
@pytest.mark.parametrize("rows", [0, 12, -1])
def test_sweeps(lda_mod, oracle_mod, K, rows):
    rng = np.random.default_rng(K)
    V = 900
    n = rng.integers(0, 9, V)
    n[:18] = [1024, 1025, 1023, 1, 0, 128, 127, 125, 126, 2048, 2049, 4097, 3, 0, 0, 1024, 900, 257]
    n[18:700] = rng.integers(0, 2, 682)  # more than 512 words to 1024 tokens
    doff, words = corpus_of(n, K)
    g = lda_mod.Lda(doff, words, V, K, 0.1, 0.01, seed=3, dense_rows=rows, dense_alias_min_count=1 << 20)
    o = oracle_mod.Oracle(doff, words, V, K, 0.1, 0.01, seed=3, dense_alias_min_count=1 << 20)
    for m in (2, 3, 1, 4, 9, 8, 2):
        for c in (g, o):
            c.build_alias(); c.sweep(m); c.rebuild_counts()
        assert np.array_equal(g.get_z(), o.get_z()), m
        assert np.array_equal(g.get_nk(), o.get_nk()), m
    for w in list(range(20)) + [700, V - 1]:
        assert np.array_equal(g.get_nkw_row(w), o.get_nkw_row(w)), w
    assert abs(g.loglik()[0] - o.loglik()[0]) <= 1e-9 * abs(o.loglik()[0])
    g.close(); o.close()


@pytest.mark.parametrize("K", [16384, 16385, 40000])
@pytest.mark.parametrize("rows,mode", [(0, 0), (200, 0), (200, 1)])
def test_rows_of_one_pass_sweeps(lda_mod, oracle_mod, K, rows, mode):
    """Sweeps of one kernel look up rows, which hold the counts of these words for the sweep alone: no
    count stays behind for the next one, in a graph's replays either."""
    import torch
    V = 900
    n = np.random.default_rng(K).integers(0, 60, V)
    n[:6] = [1024, 1025, 0, 1, 2048, 300]
    doff, words = corpus_of(n, K)
    stream = torch.cuda.Stream()
    g = lda_mod.Lda(doff, words, V, K, 0.1, 0.01, seed=3, dense_rows=rows, dense_alias_min_count=1 << 20,
                    proposal_mode=mode, stream=stream.cuda_stream)
    o = oracle_mod.Oracle(doff, words, V, K, 0.1, 0.01, seed=3, dense_alias_min_count=1 << 20, proposal_mode=mode)
    for m in (9, 9, 2, 10, 1, 9):
        for c in (g, o):
            c.build_alias(); c.sweep(m); c.rebuild_counts()
        assert np.array_equal(g.get_z(), o.get_z()), m
        for w in range(0, V, 61):
            assert np.array_equal(g.get_nkw_row(w), o.get_nkw_row(w)), (m, w)
    for c in (g, o):
        c.build_alias()
    g.sync()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        g.sweep(9)
    o.sweep(9)
    for i in range(3):
        with torch.cuda.stream(stream):
            graph.replay()
        assert np.array_equal(g.get_z(), o.get_z()), i
    for c in (g, o):
        c.rebuild_counts(); c.build_alias(); c.sweep(9)
    assert np.array_equal(g.get_z(), o.get_z())
    g.close(); o.close()
