"""Word-proposal tables at the sizes where their construction changes form (a wave, several
entries per lane, a workgroup, beyond one workgroup's LDS): every table against the oracle's,
bit for bit, with even and with very uneven weights."""
import numpy as np
import pytest

from test_gpu_hybrid import check_mixture_tables
from test_gpu_parity import check_alias

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lda_mod():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_1412_1576_amd import lda
    lda.load_library()
    return lda


def word_corpus(counts, L=300):
    """Documents of L tokens over words with the given corpus frequencies."""
    words = np.repeat(np.arange(len(counts), dtype=np.int32), counts)
    np.random.default_rng(5).shuffle(words)
    doff = np.append(np.arange(0, len(words), L), len(words)).astype(np.int64)
    return doff, words


def topics(words, K, pattern, seed):
    rng = np.random.default_rng(seed)
    z = np.empty(len(words), np.int32)
    for w in range(int(words.max()) + 1):
        at = np.flatnonzero(words == w)
        if pattern == "distinct":   # as many entries as tokens (or topics)
            z[at] = rng.permutation(np.resize(rng.permutation(K), len(at)))
        else:                       # a few topics hold most of the tokens
            z[at] = (K * rng.random(len(at)) ** 6).astype(np.int32)
    return z


@pytest.mark.parametrize("pattern", ["distinct", "skewed"])
@pytest.mark.parametrize("K", [2, 63, 64, 65, 255, 256, 257, 1023, 1024, 1025, 1537, 8191, 8192,
                               8193, 12287, 12288])
def test_dense_tables(lda_mod, oracle_mod, K, pattern):
    # frequent words (their quantised weights need a shift) down to a single token
    counts = [3 * K + 7, K, K // 2 + 1, 40, 3, 1]
    doff, words = word_corpus(counts)
    g = lda_mod.Lda(doff, words, len(counts), K, 0.1, 0.01, seed=1)
    o = oracle_mod.Oracle(doff, words, len(counts), K, 0.1, 0.01, seed=1)
    z = topics(words, K, pattern, 11)
    for m in (g, o):
        m.set_z(z, 0)
        m.rebuild_counts()
        m.build_alias()
    check_alias(g, o, range(len(counts)), tag="K = %d" % K)
    g.close()
    o.close()


SIZES = [1, 2, 15, 16, 17, 31, 32, 33, 63, 64, 65, 255, 256, 257, 1023, 1024, 1025, 2047, 2048, 2049,
         4096, 4097, 8192, 8193, 12287, 12288, 12289, 16384, 16385, 29_000]


@pytest.mark.parametrize("pattern", ["distinct", "skewed"])
@pytest.mark.parametrize("K", [12_289, 30_000])
def test_mixture_tables(lda_mod, oracle_mod, K, pattern):
    doff, words = word_corpus(SIZES)
    opt = dict(seed=2, dense_alias_min_count=1 << 27)
    g = lda_mod.Lda(doff, words, len(SIZES), K, 0.1, 0.01, dense_rows=-1, **opt)
    o = oracle_mod.Oracle(doff, words, len(SIZES), K, 0.1, 0.01, **opt)
    z = topics(words, K, pattern, 12)
    for m in (g, o):
        m.set_z(z, 0)
        m.rebuild_counts()
        m.build_alias()
    check_mixture_tables(g, o, range(len(SIZES)), tag="K = %d" % K)
    g.close()
    o.close()


@pytest.mark.parametrize("pattern", ["distinct", "skewed"])
def test_dense_tables_beyond_one_workgroup(lda_mod, oracle_mod, pattern):
    """K just above what a workgroup's LDS holds, dense tables for every word, and a larger K."""
    for K in (12_289, 40_000):
        counts = [2 * K, K // 3, 50, 1]
        doff, words = word_corpus(counts)
        g = lda_mod.Lda(doff, words, len(counts), K, 0.1, 0.01, seed=3)
        o = oracle_mod.Oracle(doff, words, len(counts), K, 0.1, 0.01, seed=3)
        z = topics(words, K, pattern, 13)
        for m in (g, o):
            m.set_z(z, 0)
            m.rebuild_counts()
            m.build_alias()
        check_alias(g, o, range(len(counts)), tag="K = %d" % K)
        g.close()
        o.close()


def two_builds(g, o, sweep_check):
    for it in range(2):
        for m in (g, o):
            m.build_alias()
        sweep_check("build %d" % it)
        for m in (g, o):
            m.sweep(2)
            m.rebuild_counts()
        assert np.array_equal(g.get_z(), o.get_z()), it
    g.close()
    o.close()


# 340 K list entries hold 339 tables of K entries: the first and the last table of every batch
def test_dense_tables_in_several_batches(lda_mod, oracle_mod):
    K, V = 12_290, 700
    doff, words = word_corpus(np.random.default_rng(3).integers(1, 12, V))
    g = lda_mod.Lda(doff, words, V, K, 0.1, 0.01, seed=6)
    o = oracle_mod.Oracle(doff, words, V, K, 0.1, 0.01, seed=6)
    two_builds(g, o, lambda tag: check_alias(g, o, [0, 1, 337, 338, 339, 340, 677, 678, 679, 698, 699], tag=tag))


def test_mixture_tables_in_several_batches(lda_mod, oracle_mod):
    """Behind dense tables, which use the same list memory."""
    K, V = 12_290, 350
    counts = [20_000, 12_500, 20_001] + [12_300] * (V - 4) + [5]
    doff, words = word_corpus(counts)
    opt = dict(seed=7, dense_alias_min_count=20_000)
    g = lda_mod.Lda(doff, words, V, K, 0.1, 0.01, dense_rows=V, **opt)
    o = oracle_mod.Oracle(doff, words, V, K, 0.1, 0.01, **opt)

    def check(tag):
        check_alias(g, o, [0, 2], tag=tag)
        check_mixture_tables(g, o, [1, 3, 4, 338, 339, 340, 341, 342, 347, 348, 349], tag=tag)

    two_builds(g, o, check)
