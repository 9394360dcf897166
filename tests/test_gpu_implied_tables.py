"""Words whose dense table is implied by a few sums: sweeps against the oracle, bit for bit, where
the form begins and ends (words of 1, 64, 256, 1024 tokens and one more, words without tokens), where
a word's sums do not fit it (topics of very uneven size, weights that need a shift), in turn
with sweeps that draw from bins, and after the incremental count update.  The form is used where
the words it suits have 2^23 bins or more together, and a word suits with at most K / 2 tokens."""
import numpy as np
import pytest

from test_gpu_parity import check_alias

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lda_mod():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_1412_1576_amd import lda
    lda.load_library()
    return lda


def corpus_of(counts, seed, L=90):
    """Documents of about L tokens over words with the given corpus frequencies."""
    words = np.repeat(np.arange(len(counts), dtype=np.int32), counts)
    np.random.default_rng(seed).shuffle(words)
    return np.append(np.arange(0, len(words), L), len(words)).astype(np.int64), words


def pair(lda_mod, oracle_mod, doff, words, V, K, beta=0.01, **opt):
    return (lda_mod.Lda(doff, words, V, K, 0.1, beta, seed=3, **opt),
            oracle_mod.Oracle(doff, words, V, K, 0.1, beta, seed=3, proposal_mode=opt.get("proposal_mode", 0)))


def step(g, o, m, update=False, tables=()):
    for c in (g, o):
        c.build_alias()
    check_alias(g, o, tables, tag="%d steps" % m)
    for c in (g, o):
        c.sweep(m)
    g.update_counts() if update else g.rebuild_counts()
    o.rebuild_counts()
    assert np.array_equal(g.get_z(), o.get_z()), m
    assert np.array_equal(g.get_nk(), o.get_nk()), m
    for w in tables:
        assert np.array_equal(g.get_nkw_row(w), o.get_nkw_row(w)), (m, w)
    if len(tables):
        assert abs(g.loglik()[0] - o.loglik()[0]) <= 1e-9 * abs(o.loglik()[0])


def frequencies(V, K, seed):
    """Few to many tokens per word, the ends of the form's ranges, words without tokens."""
    n = (1 + max(8, 20 * K / V) * np.random.default_rng(seed).pareto(1.0, V)).astype(np.int64)
    n = np.minimum(n, 6000)
    ends = [0, 0, 1, 2, 63, 64, 65, 255, 256, 257, 1023, 1024, 1025, 2047, 2048, K // 2, K // 2 + 1, 0]
    n[10:10 + len(ends)] = ends
    n[-3:] = (0, 1, 0)
    return n


# K: one topic range below and above what a thread of the shared sums handles, odd, the largest
@pytest.mark.parametrize("V,K", [(46000, 257), (12000, 1024), (6200, 2051), (3400, 4099), (1400, 12287), (1400, 12288)])
@pytest.mark.parametrize("m", [2, 3])
def test_sweeps(lda_mod, oracle_mod, V, K, m):
    n = frequencies(V, K, K)
    doff, words = corpus_of(n, K)
    g, o = pair(lda_mod, oracle_mod, doff, words, V, K, beta=1e-4)
    some = list(range(0, 30)) + [V - 2, V - 1]
    for it in range(3):
        step(g, o, m, tables=some)
    g.close(); o.close()


# a topic size that varies by powers: bins without tokens are heavies for the rarer words
@pytest.mark.parametrize("power", [2, 6])
@pytest.mark.parametrize("beta", [1e-6, 0.01, 3.0])
def test_uneven_topics(lda_mod, oracle_mod, power, beta):
    V, K = 24000, 1024
    doff, words = corpus_of(frequencies(V, K, 8), 8)
    g, o = pair(lda_mod, oracle_mod, doff, words, V, K, beta=beta)
    z = (K * np.random.default_rng(4).random(len(words)) ** power).astype(np.int32)
    for c in (g, o):
        c.set_z(z, 7)
        c.rebuild_counts()
    for m in (2, 1, 4):
        step(g, o, m, tables=range(0, V, 397))
    g.close(); o.close()


def test_few_tokens(lda_mod, oracle_mod):
    """Some words have a share of the corpus so large that their weights need a shift."""
    V, K = 2600, 4001
    n = np.full(V, 27) + np.arange(V) // 120
    n[100:140] = np.linspace(150, 1024, 40).astype(int)
    doff, words = corpus_of(n, 2, L=7)
    g, o = pair(lda_mod, oracle_mod, doff, words, V, K, beta=1e-5)
    for m in (2, 4, 2):
        step(g, o, m, tables=(0, 100, 110, 139, 599))
    g.close(); o.close()


def test_in_turn_with_one_pass_sweeps(lda_mod, oracle_mod):
    V, K = 12000, 1024
    doff, words = corpus_of(frequencies(V, K, 5), 5)
    g, o = pair(lda_mod, oracle_mod, doff, words, V, K, beta=1e-4)
    for m in (2, 9, 9, 2, 4, 10, 2, 2):
        step(g, o, m, tables=(5, 13, 1000))
    g.close(); o.close()


@pytest.mark.parametrize("update", [False, True])
def test_back_to_implied_tables(lda_mod, oracle_mod, update):
    """Two-pass sweeps after a one-pass sweep: four that draw from bins, then from implied tables again."""
    V, K = 12000, 1024
    doff, words = corpus_of(frequencies(V, K, 5), 5)
    g, o = pair(lda_mod, oracle_mod, doff, words, V, K, beta=1e-4, record_bucket_tokens=4096)
    for i, m in enumerate((9, 2, 4, 1, 2, 2, 2, 9, 3, 10, 2, 2, 2, 2, 2, 2)):
        step(g, o, m, update=update and i in (3, 6, 12), tables=(0, 5, 13, 1000))
    g.close(); o.close()


def test_words_without_tokens_in_used_memory(lda_mod, oracle_mod):
    """The first sweep of a new sampler is one kernel, which draws from bins, and the caller's memory
    has been used before: the rows that the bins of words without tokens are made from are zero."""
    import torch
    V, K = 12000, 1024
    n = frequencies(V, K, 5)
    empty = [0, 1, 2, V // 2, V - 2, V - 1]
    n[empty] = 0
    doff, words = corpus_of(n, 5)
    live = {}

    def alloc(nbytes):
        t = torch.full((nbytes,), 0x3b, dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        live[t.data_ptr()] = t
        return t.data_ptr()

    g, o = pair(lda_mod, oracle_mod, doff, words, V, K, beta=1e-4, dev_alloc=alloc, dev_free=lambda p: live.pop(p))

    def array(counts):
        t, = [t for t in live.values() if t.numel() == 4 * counts]
        return t.view(torch.int32)

    # before any kernel reads them
    assert not array(V * K).view(V, K)[torch.tensor(empty, device="cuda")].any()
    o.build_alias()
    split, alias, cap = zip(*[o.get_alias_row(w) for w in empty])
    g.build_alias(); g.sweep(9); o.sweep(9)
    g.sync()
    bins = array(V * K * 4).view(V, K, 4)[torch.tensor(empty, device="cuda")].cpu().numpy()
    assert np.array_equal(bins[:, :, 0].view(np.uint32), np.stack(split))
    assert np.array_equal(bins[:, :, 1].view(np.uint32), np.stack(alias))
    assert not bins[:, :, 2:].any()
    g.rebuild_counts(); o.rebuild_counts()
    for m in (2, 9, 2):
        step(g, o, m, tables=empty + [5, 13])
    g.close(); o.close()
    assert not live


def test_after_the_incremental_update(lda_mod, oracle_mod):
    V, K = 36000, 300
    doff, words = corpus_of(frequencies(V, K, 6), 6, L=12)
    for turns in ("uuu", "ruurrrru"):  # rows are kept for updates, lists for recounts
        g, o = pair(lda_mod, oracle_mod, doff, words, V, K)
        for i, turn in enumerate(turns):
            step(g, o, 9 if i == 4 else 2 + i % 2, update=turn == "u", tables=(5, 13, 8000))
        g.close(); o.close()


def test_few_moved_tokens(lda_mod, oracle_mod):
    """One token moved since the recount: the incremental update finds the rows stale and counts."""
    V, K = 12000, 1024
    doff, words = corpus_of(frequencies(V, K, 7), 7)
    g, o = pair(lda_mod, oracle_mod, doff, words, V, K, proposal_mode=1, beta=1e-9)
    z = words % K  # every word in one topic, which its proposals hardly leave
    for c in (g, o):
        c.set_z(z, 0)
        c.rebuild_counts()
    for update in (True, True, False, True):
        step(g, o, 1, update=update, tables=range(0, V, 411))
    g.close(); o.close()


def test_graph_replays_leave_lists(lda_mod, oracle_mod):
    """What the rows hold is known on the device: iterations replayed from a graph leave lists where
    the host, which saw an update before, would expect rows."""
    import torch
    V, K = 12000, 1024
    doff, words = corpus_of(frequencies(V, K, 3), 3)
    stream = torch.cuda.Stream()
    g = lda_mod.Lda(doff, words, V, K, 0.1, 1e-4, seed=3, stream=stream.cuda_stream)
    for _ in range(2):
        g.build_alias(); g.sweep(2); g.rebuild_counts()
    g.sync()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        g.rebuild_counts()
    g.build_alias(); g.sweep(2); g.update_counts()
    g.build_alias(); g.sweep(2); g.update_counts()
    z = g.get_z()
    with torch.cuda.stream(stream):
        for _ in range(3):
            graph.replay()
    g.sync()
    rows = np.zeros((V, K), np.int32)
    np.add.at(rows, (words, z), 1)
    for w in range(0, V, 137):
        assert np.array_equal(g.get_nkw_row(w), rows[w]), w
    g.build_alias(); g.sweep(2); g.update_counts()
    z = g.get_z()
    rows[:] = 0
    np.add.at(rows, (words, z), 1)
    for w in range(0, V, 137):
        assert np.array_equal(g.get_nkw_row(w), rows[w]), w
    g.close()


@pytest.mark.parametrize("captured,others", [(2, (9,)), (9, (2, 2, 2, 2, 2))])
def test_a_captured_sweep_finds_its_tables(lda_mod, oracle_mod, captured, others):
    """A graph of a sweep and its recount, replayed after builds that the host made between sweeps that
    draw from the other form of the tables."""
    import torch
    V, K = 12000, 1024
    doff, words = corpus_of(frequencies(V, K, 4), 4)
    stream = torch.cuda.Stream()
    g, o = pair(lda_mod, oracle_mod, doff, words, V, K, beta=1e-4, stream=stream.cuda_stream)
    g.build_alias(); g.sweep(2)  # takes the records, which a capture cannot
    z = np.random.default_rng(1).integers(0, K, len(words)).astype(np.int32)
    g.set_z(z, 7)
    g.rebuild_counts(); g.build_alias(); g.sync()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        g.sweep(captured)  # reads the one array of assignments and writes the other
        g.rebuild_counts()
    with torch.cuda.stream(stream):
        graph.replay()
    for m in others:  # an odd number: back into the one that the graph reads
        g.build_alias(); g.sweep(m); g.rebuild_counts()
    o.set_z(g.get_z(), 7)
    o.rebuild_counts(); o.build_alias(); g.build_alias()
    o.sweep(captured); o.rebuild_counts()
    with torch.cuda.stream(stream):
        graph.replay()
    assert np.array_equal(g.get_nk(), o.get_nk())
    for w in range(0, V, 411):
        assert np.array_equal(g.get_nkw_row(w), o.get_nkw_row(w)), w
    g.close(); o.close()


def test_record_order_and_word_chains(lda_mod, oracle_mod):
    V, K = 12000, 1024
    doff, words = corpus_of(frequencies(V, K, 9), 9)
    g, o = pair(lda_mod, oracle_mod, doff, words, V, K, beta=1e-4, record_bucket_tokens=4096)
    for m in (2, 4):
        step(g, o, m)
    g.close(); o.close()
    g = lda_mod.Lda(doff, words, V, K, 0.1, 1e-4, seed=3, proposal_mode=1)
    o = oracle_mod.Oracle(doff, words, V, K, 0.1, 1e-4, seed=3, proposal_mode=1)
    for m in (1, 3, 1, 1):
        step(g, o, m)
    g.close(); o.close()


@pytest.mark.parametrize("V", [40, 12000])
def test_a_failed_build_leaves_no_tables(lda_mod, oracle_mod, V):
    """The library reports an error that an earlier HIP call of the thread left; no table is given out
    or drawn from until they are built again."""
    K = 1024
    doff, words = corpus_of(np.full(V, 40), 4)
    g, o = pair(lda_mod, oracle_mod, doff, words, V, K)
    g.build_alias(); o.build_alias()
    assert lda_mod.load_library().hipSetDevice(999) != 0
    with pytest.raises(lda_mod.LdaError) as e:
        g.build_alias()
    assert e.value.code == lda_mod.LDA_ERR_HIP
    for call in (lambda: g.get_alias_row(3), lambda: g.sweep(2)):
        with pytest.raises(lda_mod.LdaError) as e:
            call()
        assert e.value.code == lda_mod.LDA_ERR_STATE
    step(g, o, 2, tables=(0, 3))
    g.close(); o.close()


class Pool:
    """A caller's allocator that refuses requests beyond a number of them, or of bytes held."""
    def __init__(self, requests=1 << 60, most=1 << 60):
        self.live, self.requests, self.left, self.most = {}, 0, requests, most

    def held(self):
        return sum(t.numel() for t in self.live.values())

    def alloc(self, nbytes):
        import torch
        self.requests += 1
        if self.requests > self.left or self.held() + nbytes > self.most:
            return 0
        t = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        self.live[t.data_ptr()] = t
        return t.data_ptr()

    def options(self):
        return {"dev_alloc": self.alloc, "dev_free": lambda p: self.live.pop(p)}


def test_without_room_for_the_lists(lda_mod, oracle_mod):
    """An allocator that fails at the last, the last but one, ... request of lda_init: as long as what a
    sampler cannot do without is there, every word has its bins."""
    V, K = 12000, 1024
    doff, words = corpus_of(frequencies(V, K, 5), 5)
    all_of_it = Pool()
    pair(lda_mod, oracle_mod, doff, words, V, K, beta=1e-4, **all_of_it.options())[0].close()
    without = []
    for left in range(all_of_it.requests - 1, 0, -1):
        pool = Pool(requests=left)
        try:
            g, o = pair(lda_mod, oracle_mod, doff, words, V, K, beta=1e-4, **pool.options())
        except lda_mod.LdaError as e:
            assert e.code == lda_mod.LDA_ERR_OOM and not pool.live
            break
        without.append(pool.held())
        pool.left = 1 << 60
        if len(without) in (1, 9):
            for i, m in enumerate((2, 9, 2, 4)):
                step(g, o, m, update=i == 2, tables=(0, 5, 13, 1000))
        g.close(); o.close()
        assert not pool.live
    assert len(without) > 9 and len(set(without)) == 1


@pytest.mark.parametrize("captured", [False, True])
def test_records_take_the_room_of_the_lists(lda_mod, oracle_mod, captured):
    """A sweep that finds no room for its records beside the lists, and does without them; not where
    a graph may replay work that uses the lists."""
    import torch
    V, K = 12000, 1024
    doff, words = corpus_of(frequencies(V, K, 5), 5)
    stream = torch.cuda.Stream()
    pool = Pool()
    g, o = pair(lda_mod, oracle_mod, doff, words, V, K, beta=1e-4, stream=stream.cuda_stream, **pool.options())
    pool.left = pool.requests
    lists, n = pool.held(), pool.requests
    g.close()
    pool = Pool(requests=n - 1)
    g = lda_mod.Lda(doff, words, V, K, 0.1, 1e-4, seed=3, stream=stream.cuda_stream, **pool.options())
    bins = pool.held()
    g.close()
    records = 16 * len(words)
    assert lists - bins > 1 << 18
    pool = Pool(most=bins + records + (1 << 16))
    g = lda_mod.Lda(doff, words, V, K, 0.1, 1e-4, seed=3, stream=stream.cuda_stream, **pool.options())
    assert pool.held() == lists
    if captured:
        g.sync()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            g.rebuild_counts()
        g.build_alias()
        with pytest.raises(lda_mod.LdaError) as e:
            g.sweep(2)
        assert e.value.code == lda_mod.LDA_ERR_OOM and pool.held() == lists
        g.rebuild_counts()
        pool.most = 1 << 60
    for i, m in enumerate((2, 2, 9, 2)):
        step(g, o, m, update=i == 1, tables=(0, 5, 13, 1000))
    assert captured or pool.held() <= pool.most
    pool.most = 1 << 60
    step(g, o, 4, tables=(0, 5, 13, 1000))
    g.close(); o.close()
    assert not pool.live
