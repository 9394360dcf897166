"""Count rebuild with thousands of short words, each counted by one wave, beside words that take a
workgroup; against the oracle."""
import numpy as np
import pytest

from test_gpu_hybrid import check_mixture_tables
from test_gpu_parity import check_state

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lda_mod():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_1412_1576_amd import lda
    lda.load_library()
    return lda


# words of 512 tokens are a wave's, of 513 a workgroup's; K up to 2048 takes waves, from 2049 none
@pytest.mark.parametrize("K,min_count,bucket", [(1, 0, 0), (65, 0, 0), (2048, 600, 0), (2049, 600, 0),
                                                (130, 130, 1024)])
def test_rows_lists_and_updates(lda_mod, oracle_mod, K, min_count, bucket):
    rng = np.random.default_rng(K)
    counts = np.concatenate([[3000, 513, 512, 511, 601, 600, 599, 129, 128, 127, 65, 64, 63, 0],
                             rng.integers(0, 9, 4200)])
    V = len(counts)
    words = np.repeat(np.arange(V), counts).astype(np.int32)
    rng.shuffle(words)
    doff = np.append(np.arange(0, len(words), 57), len(words)).astype(np.int64)
    opt = {"dense_alias_min_count": min_count} if min_count else {}
    g = lda_mod.Lda(doff, words, V, K, 0.1, 0.01, seed=2, record_bucket_tokens=bucket, **opt)
    o = oracle_mod.Oracle(doff, words, V, K, 0.1, 0.01, seed=2, **opt)
    rows = list(range(16)) + list(range(16, V, 61)) + [V - 1]
    for it in range(3):
        g.build_alias(); o.build_alias()
        if min_count:
            check_mixture_tables(g, o, [w for w in rows if counts[w] < min_count])
        g.sweep(2); o.sweep(2)
        if it == 1 and not min_count:
            g.update_counts()
        else:
            g.rebuild_counts()
        o.rebuild_counts()
        check_state(g, o, words=rows, tag="sweep %d" % it)
    g.close(); o.close()
