"""lda_update_counts on both sides of its rule: few moved tokens are applied one by one, many make
it recount, and a small corpus never asks.  The counts are the oracle's either way."""
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


# (tokens, V, K, steps of each sweep): 4 * 10^5 tokens ask the sample, whose line is at about half
# of them moved -- nearly all move with K = 300, few with K = 2; a sweep of 9 steps leaves no
# word-major copy of the assignment behind, which the recount then has to make
@pytest.mark.parametrize("N,V,K,steps", [(400_001, 50, 300, (2, 2, 9)), (400_001, 50, 2, (2, 9, 2)),
                                         (400_001, 700, 65, (1, 9, 9, 2)), (3_001, 50, 300, (2, 9)),
                                         (400_001, 50, 300, (5, 8)), (400_001, 50, 300, (9, 2, 2))])
def test_update_equals_recount(lda_mod, oracle_mod, N, V, K, steps):
    rng = np.random.default_rng(7)
    words = (V * rng.random(N) ** 3).astype(np.int32)
    doff = np.append(np.arange(0, N, 90), N).astype(np.int64)
    g = lda_mod.Lda(doff, words, V, K, 0.1, 0.01, seed=4)
    o = oracle_mod.Oracle(doff, words, V, K, 0.1, 0.01, seed=4)
    for i, mh in enumerate(steps):
        for m in (g, o):
            m.build_alias()
            m.sweep(mh)
        g.update_counts()
        o.rebuild_counts()
        assert np.array_equal(g.get_z(), o.get_z()), "sweep %d" % i
        assert np.array_equal(g.get_nk(), o.get_nk()), "n_k after sweep %d" % i
        for w in range(V):
            assert np.array_equal(g.get_nkw_row(w), o.get_nkw_row(w)), "word %d, sweep %d" % (w, i)
    g.close()
    o.close()


# more tiles than the workgroups of a recount that may not be wanted: of a workgroup each (K above
# 2048, then an LDS histogram of 48 KB), and of a wave each (four to a workgroup)
@pytest.mark.parametrize("V,K", [(8400, 2049), (8400, 12_288), (34_000, 70)])
@pytest.mark.parametrize("steps", [2, 9])
def test_many_tiles_wanted_or_not(lda_mod, oracle_mod, V, K, steps):
    rng = np.random.default_rng(V + K)
    N = 3_000_000
    words = (V * rng.random(N) ** 2).astype(np.int32)
    words[:V] = np.arange(V)
    doff = np.append(np.arange(0, N, 90), N).astype(np.int64)
    g = lda_mod.Lda(doff, words, V, K, 1e-5, 0.01, seed=4)
    z = rng.integers(0, K, N).astype(np.int32)
    # the line lies between 16 and 50 % of the tokens: most move; then hardly any does, with one topic
    # to every word and document
    for zz, moves in ((z, True), (np.zeros(N, np.int32), False), (z, True)):
        g.set_z(zz, 3)
        g.rebuild_counts()
        g.build_alias()
        g.sweep(steps)
        after = g.get_z()
        share = float((after != zz).mean())
        assert share > 0.5 if moves else share < 0.05, share
        g.update_counts()
        nk, rows = g.get_nk(), [g.get_nkw_row(w) for w in range(0, V, 83)]
        assert np.array_equal(nk, np.bincount(after, minlength=K))
        for w, row in zip(range(0, V, 83), rows):
            assert np.array_equal(row, np.bincount(after[words == w], minlength=K)), w
        g.rebuild_counts()  # and every row, by the recount
        assert np.array_equal(g.get_nk(), nk)
    g.close()


# the refreshed sweep leaves no word-major copy either: nearly all tokens move, then about half
@pytest.mark.parametrize("V,K", [(50, 300), (50, 2), (9_000, 65)])
def test_after_refreshed_sweeps(lda_mod, oracle_mod, V, K):
    rng = np.random.default_rng(V + K)
    N = 400_001
    words = (V * rng.random(N) ** 3).astype(np.int32)
    doff = np.append(np.arange(0, N, 90), N).astype(np.int64)
    g = lda_mod.Lda(doff, words, V, K, 0.1, 0.01, seed=4, doc_refresh=1)
    o = oracle_mod.Oracle(doff, words, V, K, 0.1, 0.01, seed=4)
    for i, (mh, update) in enumerate([(2, True), (2, True), (3, False), (1, True)]):
        g.build_alias(); o.build_alias()
        g.sweep(mh); o.sweep_doc_refresh(mh)
        if update:
            g.update_counts()
        else:
            g.rebuild_counts()
        o.rebuild_counts()
        assert np.array_equal(g.get_z(), o.get_z()), i
        assert np.array_equal(g.get_nk(), o.get_nk()), i
        for w in range(0, V, max(1, V // 150)):
            assert np.array_equal(g.get_nkw_row(w), o.get_nkw_row(w)), (i, w)
    g.close()
    o.close()
