"""The log-likelihood on both sides of its table of terms (counts below and from 4096 on, of words
and of documents), against the oracle; the allocation-free form returns the same bits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 3])
@pytest.mark.parametrize("n", [4095, 4096, 4097, 20_000])
def test_counts_around_the_table(oracle_mod, K, n):
    from paper_1412_1576_amd import lda
    words = np.concatenate([np.zeros(n, np.int32), np.arange(1, 40, dtype=np.int32)])
    doff = np.array([0, n, n + 3, len(words)], np.int64)  # a document of n tokens of one word
    g = lda.Lda(doff, words, 40, K, 0.1, 0.01, seed=3)
    o = oracle_mod.Oracle(doff, words, 40, K, 0.1, 0.01, seed=3)
    got, want = g.loglik(), o.loglik()
    # 1e-9 relative to the terms, which can cancel: the bound of the other log-likelihood tests
    for a, b in zip(got, want):
        assert abs(a - b) <= 1e-9 * max(abs(b), abs(want[0])) + 2e-7, (K, n, got, want)
    assert g.loglik_noalloc() == got
    g.close()
    o.close()


@pytest.mark.parametrize("K", [1, 64, 511, 513, 4095, 4096, 4097, 4609, 8192, 8300])
def test_rows_beside_lists(oracle_mod, K):
    """Rows in pieces of 4096 counts, read 512 at a time, in a store whose other words have lists."""
    from paper_1412_1576_amd import lda
    counts = np.random.default_rng(K).integers(0, 40, 60)
    counts[[0, 3, 59]] = [8300, 9001, 8301]  # dense tables, and so rows
    words = np.repeat(np.arange(60, dtype=np.int32), counts)
    np.random.default_rng(K + 1).shuffle(words)
    doff = np.append(np.arange(0, len(words), 90), len(words)).astype(np.int64)
    g = lda.Lda(doff, words, 60, K, 0.1, 0.01, seed=3, dense_alias_min_count=8300)
    o = oracle_mod.Oracle(doff, words, 60, K, 0.1, 0.01, seed=3, dense_alias_min_count=8300)
    for sweep in range(2):
        got, want = g.loglik(), o.loglik()
        for a, b in zip(got, want):
            assert abs(a - b) <= 1e-9 * max(abs(b), abs(want[0])) + 2e-7, (K, sweep, got, want)
        assert g.loglik_noalloc() == got
        for c in (g, o):
            c.build_alias(); c.sweep(2); c.rebuild_counts()
    g.close()
    o.close()
