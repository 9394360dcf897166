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
# of them moved -- nearly all move with K = 300, few with K = 2; 5 steps leave no word-major copy
# of the assignment behind, which the recount then has to make
@pytest.mark.parametrize("N,V,K,steps", [(400_001, 50, 300, (2, 2, 5)), (400_001, 50, 2, (2, 5, 2)),
                                         (400_001, 700, 65, (1, 5, 5, 2)), (3_001, 50, 300, (2, 5))])
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
