"""Doc pass against the oracle, bit for bit, where its forms meet: counters per document or hash tables
(K around what fits a tile), the 32-bit accept test with its margin and the 64-bit one it leaves the
rest to (alpha and beta from ordinary to where the 32-bit products could leave their range), and doc
proposals that all but never or always copy a token."""
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


def make(lens, V, seed):
    rng = np.random.default_rng(seed)
    doff = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    p = 1.0 / np.arange(1, V + 1)
    return doff, rng.choice(V, int(doff[-1]), p=p / p.sum()).astype(np.int32)


def check(lda_mod, oracle_mod, doff, words, V, K, alpha, beta, steps, **opt):
    g = lda_mod.Lda(doff, words, V, K, alpha, beta, seed=2, **opt)
    o = oracle_mod.Oracle(doff, words, V, K, alpha, beta, seed=2)
    for m in steps:
        for c in (g, o):
            c.build_alias(); c.sweep(m); c.rebuild_counts()
        assert np.array_equal(g.get_z(), o.get_z()), (K, alpha, beta, m)
        assert np.array_equal(g.get_nk(), o.get_nk())
    for d in (0, len(doff) - 2):
        assert np.array_equal(g.get_ndk_row(d), o.get_ndk_row(d))
    g.close(); o.close()


# documents of about 1000 tokens: one document's K counters fill the room of a tile at 6144 topics
# (1536 tokens) and 4096 (1024 tokens, longer chains); short documents keep their hash tables
@pytest.mark.parametrize("K", [1, 2, 3, 255, 4095, 4096, 4097, 6143, 6144, 6145])
@pytest.mark.parametrize("L", [1000, 40])
def test_tables_of_a_document(lda_mod, oracle_mod, K, L):
    rng = np.random.default_rng(K)
    lens = np.concatenate([[0, 1, L, 1024, 0], rng.integers(L - L // 8, L + L // 8, 30000 // L), [1023, 2, 0]])
    doff, words = make(lens, 60, K)
    check(lda_mod, oracle_mod, doff, words, 60, K, 0.1, 0.01, (2, 3, 2))


@pytest.mark.parametrize("tile,block", [(64, 64), (512, 256), (1024, 1024), (1984, 512)])
def test_other_tiles(lda_mod, oracle_mod, tile, block):
    lens = np.concatenate([[63, 64, 0, 65], np.random.default_rng(tile).integers(0, 300, 60), [tile, tile + 1]])
    doff, words = make(lens, 60, tile)
    check(lda_mod, oracle_mod, doff, words, 60, 200, 0.1, 0.01, (2, 4, 1), sweep_chunk_tokens=tile,
          sweep_block_threads=block)


@pytest.mark.parametrize("alpha,beta", [(1e-12, 1e-12), (1e-30, 0.01), (0.1, 1e-30), (1e-30, 1e-30), (1e-200, 1e-100),
                                        (50.0, 20.0), (1e8, 1e8), (1e30, 1e30), (1e12, 0.01), (1e-9, 1e9)])
@pytest.mark.parametrize("K", [50, 3000])
def test_range_of_alpha_and_beta(lda_mod, oracle_mod, alpha, beta, K):
    lens = np.concatenate([np.random.default_rng(K).integers(1, 200, 80), [1500, 5]])
    doff, words = make(lens, 90, K)
    check(lda_mod, oracle_mod, doff, words, 90, K, alpha, beta, (2, 4, 2, 8, 2))


# documents beyond a tile: counters in LDS up to 32 768 topics, slices of 1024 tokens and, beyond 64 of
# them, longer ones
@pytest.mark.parametrize("K", [1, 40, 32768, 32769])
def test_long_documents(lda_mod, oracle_mod, K):
    doff, words = make([1025, 70001, 0, 2048, 3, 2049, 66000, 5000], 40, K)
    g = lda_mod.Lda(doff, words, 40, K, 0.1, 0.01, seed=2)
    o = oracle_mod.Oracle(doff, words, 40, K, 0.1, 0.01, seed=2)
    for m in (2, 2, 3, 1, 4):
        for c in (g, o):
            c.build_alias(); c.sweep(m); c.rebuild_counts()
        assert np.array_equal(g.get_z(), o.get_z()), m
    a, b = g.loglik(), o.loglik()
    assert abs(a[0] - b[0]) <= 1e-9 * max(abs(b[0]), 1e6) and g.loglik()[0] == g.loglik_noalloc()[0] == a[0]
    g.close(); o.close()


# slices longer than 1024 tokens because there are many long documents, and one far longer than the others
@pytest.mark.parametrize("K", [40, 4099])
def test_many_long_documents(lda_mod, oracle_mod, K):
    lens = np.concatenate([np.random.default_rng(K).integers(1000, 2060, 800), [70001, 1024, 1025, 0, 2048, 2049, 5]])
    assert lens[lens > 1024].sum() > 1024 * 1024
    doff, words = make(lens, 40, K)
    check(lda_mod, oracle_mod, doff, words, 40, K, 0.1, 0.01, (2, 4, 2))
