"""lda_options.doc_refresh: the sweep that refreshes the doc side after every token (Sec. 4.2,
footnote 4) against the oracle's ldaref_sweep_doc_refresh, bit for bit."""
import numpy as np
import pytest

from paper_1412_1576_amd import corpus

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lda_mod():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_1412_1576_amd import lda
    lda.load_library()
    return lda


def run(lda_mod, oracle_mod, doff, words, V, K, alpha, beta, steps, mode=0, seed=3):
    g = lda_mod.Lda(doff, words, V, K, alpha, beta, seed=seed, proposal_mode=mode, doc_refresh=1)
    o = oracle_mod.Oracle(doff, words, V, K, alpha, beta, seed=seed, proposal_mode=mode)
    for it, m in enumerate(steps):
        g.build_alias(); o.build_alias()
        g.sweep(m); o.sweep_doc_refresh(m)
        g.rebuild_counts(); o.rebuild_counts()
        zg, zo = g.get_z(), o.get_z()
        assert np.array_equal(zg, zo), (it, m, int((zg != zo).sum()), len(zg))
        assert np.array_equal(g.get_nk(), o.get_nk()), (it, m)
    lg, lo = g.loglik(), o.loglik()
    assert abs(lg[0] - lo[0]) <= 1e-9 * abs(lo[0])
    g.close(); o.close()


def test_c1_every_sweep(lda_mod, oracle_mod):
    cfg = corpus.CONFIGS["c1"]
    doff, words = corpus.make_corpus(cfg)
    run(lda_mod, oracle_mod, doff, words, cfg.V, cfg.K, cfg.alpha, cfg.beta, [2] * 6 + [4, 1, 3, 2])


def test_ragged_documents_modes_and_K(lda_mod, oracle_mod):
    rng = np.random.default_rng(8)
    # empty documents first, last and in between; one-token documents; documents of 63, 64, 65,
    # 128, 129 and 4096 tokens (the limit: 64 rounds of 64 turns)
    lens = np.array([0, 1, 63, 0, 64, 65, 1, 128, 129, 7, 4096, 2, 0, 300, 0])
    doff = np.zeros(len(lens) + 1, np.int64)
    doff[1:] = np.cumsum(lens)
    for V, K in ((50, 1), (50, 2), (300, 65), (300, 3000)):
        words = rng.integers(0, V, doff[-1]).astype(np.int32)
        for mode in (0, 1, 2):
            run(lda_mod, oracle_mod, doff, words, V, K, 0.1, 0.01, [2, 3, 1, 4], mode=mode, seed=V + mode)


# lanes to a document: 8 up to K = 1200 or so at these lengths, then 16, 32, 64; beyond 256
# counters per token of a mean document (24 tokens) no counters; fewer documents take more lanes
@pytest.mark.parametrize("K,D", [(1, 4200), (7, 4200), (1000, 4200), (1001, 2100), (1300, 4200),
                                 (3000, 4200), (6001, 4200), (6300, 4200), (33, 100)])
def test_every_number_of_lanes(lda_mod, oracle_mod, K, D):
    rng = np.random.default_rng(K)
    lens = rng.integers(0, 49, D)
    lens[:12] = (0, 7, 8, 9, 15, 16, 17, 31, 32, 33, 64, 65)
    doff = np.zeros(D + 1, np.int64)
    doff[1:] = np.cumsum(lens)
    V = 61
    words = rng.integers(0, V, doff[-1]).astype(np.int32)
    run(lda_mod, oracle_mod, doff, words, V, K, 0.1, 0.01, [2, 4])
    run(lda_mod, oracle_mod, doff, words, V, K, 0.1, 0.01, [3], mode=2)


def test_what_the_mode_refuses(lda_mod):
    cfg = corpus.scaled(corpus.CONFIGS["c1"], D=50)
    doff, words = corpus.make_corpus(cfg)
    with pytest.raises(lda_mod.LdaError) as e:     # lists and hash rows: not with this sweep
        lda_mod.Lda(doff, words, cfg.V, cfg.K, cfg.alpha, cfg.beta, doc_refresh=1,
                    dense_alias_min_count=cfg.K)
    assert e.value.code == lda_mod.LDA_ERR_UNSUPPORTED
    long_doff = np.array([0, 4097], np.int64)
    with pytest.raises(lda_mod.LdaError) as e:
        lda_mod.Lda(long_doff, np.zeros(4097, np.int32), 4, 8, 0.1, 0.1, doc_refresh=1)
    assert e.value.code == lda_mod.LDA_ERR_UNSUPPORTED
    g = lda_mod.Lda(doff, words, cfg.V, cfg.K, cfg.alpha, cfg.beta, doc_refresh=1)
    g.build_alias()
    with pytest.raises(lda_mod.LdaError) as e:
        g.sweep(5)
    assert e.value.code == lda_mod.LDA_ERR_UNSUPPORTED
    g.close()


def test_refresh_against_snapshot_on_planted_topics(lda_mod):
    """Both sweeps raise the likelihood of the planted-topic corpus; the refreshed doc side
    is the less stale of the two (reported in the design notes, not asserted as a ranking)."""
    cfg = corpus.scaled(corpus.CONFIGS["c1"], D=600)
    doff, words = corpus.make_corpus(cfg)
    out = {}
    for refresh in (0, 1):
        g = lda_mod.Lda(doff, words, cfg.V, cfg.K, cfg.alpha, cfg.beta, seed=1, doc_refresh=refresh)
        ll = [g.loglik()[0]]
        for it in range(30):
            g.build_alias(); g.sweep(2); g.rebuild_counts()
            ll.append(g.loglik()[0])
        out[refresh] = ll
        g.close()
        assert ll[-1] > ll[0] and ll[10] > ll[0]
    print("loglik after 5/10/30 sweeps: snapshot %.5e %.5e %.5e, doc refresh %.5e %.5e %.5e"
          % (out[0][5], out[0][10], out[0][30], out[1][5], out[1][10], out[1][30]))
