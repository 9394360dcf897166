"""Workloads of the LightLDA sampler that its speed is judged on.

A pass is what a training program does between two checkpoints: some iterations of
{alias tables, Metropolis-Hastings sweep, counts}, the log-likelihood when the program
watches it, and the assignment and topic totals copied out into the program's own buffers.
The corpora are the seeded synthetic ones of the package (Zipf words, Poisson lengths,
planted topics where the workload has them).
"""
import math
from dataclasses import replace

import numpy as np
import torch

from paper_1412_1576_amd import corpus, lda


def _case(name, base, iters, mh=2, store="dense", docs=0, ragged=False, K=0, V=0, lam=0.0,
          T=-1, dense_rows=0, refresh=False, update=False, block=0, loglik_every=0):
    """A case from one of the package's workload configurations and what it changes of it."""
    c = corpus.CONFIGS[base]
    case = {"D": docs or c.D, "lam": float(lam or c.lam), "ragged": ragged, "V": V or c.V, "s": c.s,
            "T": c.T if T < 0 else T, "K": K or c.K, "alpha": c.alpha, "beta": c.beta, "mh": mh,
            "iters": iters, "store": store, "dense_rows": dense_rows, "refresh": refresh,
            "update": update, "block": block, "loglik_every": loglik_every}
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # a first experiment: 10^5 tokens, library defaults (a dense table for every word), ten
        # sweeps with one look at the likelihood; some ten launches a sweep decide it
        _case("tiny_10_sweeps", "c1", iters=10, loglik_every=10),
        # a small collection of very uneven documents (empty ones, and some beyond every tile),
        # an odd number of topics, three-step chains
        _case("ragged_3_steps", "c1", iters=5, mh=3, store="mixture", docs=401, ragged=True, K=257,
              V=2999, lam=180, loglik_every=5),
        # a collection of a few million tokens trained while the likelihood is watched
        _case("watched_loglik", "c2", iters=5, store="mixture", docs=11_269, lam=170, V=53_975, T=20,
              K=500, loglik_every=1),
        # messages: very short documents, counts kept by the paper's own +-1 rule
        _case("short_docs_update", "c1", iters=5, docs=150_001, lam=12, V=30_011, K=333, update=True),
        # the NYTimes-shaped corpus, whole, with the proposal form the benchmark uses
        _case("nytimes_k1000", "c2", iters=20, store="mixture"),
        # a fifth of it with long chains, the paper's way to more progress per sweep
        _case("nytimes_8_steps", "c2", iters=2, mh=8, store="mixture", docs=60_000),
        # a fifth of it with the doc side refreshed after every token (Sec. 4.2, footnote 4)
        _case("nytimes_refresh", "c2", iters=2, docs=60_000, refresh=True, loglik_every=2),
        # the PubMed-shaped corpus, whole: the headline workload
        _case("pubmed_k10000", "c3", iters=20, store="mixture"),
        # a part of it under the configuration's own settings: four steps, dense tables throughout
        _case("pubmed_4_steps_dense", "c3", iters=5, mh=4, docs=600_000),
        # K = 10^5: dense rows for the head words, lists and hash rows for the tail
        _case("hybrid_k100000", "c4", iters=3, store="hybrid", docs=1_500_000, dense_rows=20_000),
        # one K = 10^6 slice: every word a list and a hash row
        _case("sparse_k1000000", "c5", iters=3, store="hybrid", docs=1_000_000, dense_rows=-1),
        # the same with the corpus in host memory, passing through the GPU in blocks
        _case("streamed_k1000000", "c5", iters=3, store="hybrid", docs=400_000, dense_rows=-1,
              block=10_000_000),
    ]


def draw(rng):
    def spread(lo, hi):  # over the logarithm, odd sizes included
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    family = rng.choice(("dense", "dense", "mixture", "mixture", "steps", "refresh", "hybrid",
                         "sparse", "streamed"))
    lam = float(spread(8, 400))
    most = {"dense": 5e7, "mixture": 2e8, "steps": 2e7, "refresh": 2e7, "hybrid": 1e8,
            "sparse": 6e7, "streamed": 4e7}[family]
    docs = max(20, spread(3e4, most) // int(lam))
    base = rng.choice(("c1", "c2", "c3"))
    T = rng.choice((0, 20, 200))
    ragged = rng.random() < 0.25 and family != "streamed"
    iters = rng.randint(1, 6)
    mh = rng.choice((1, 2, 2, 2, 3, 4))
    V = spread(2_000, 150_000)
    if family in ("dense", "refresh"):
        K = spread(30, min(12_000, 4e8 / V))
        refresh = family == "refresh"
        return _case("", base, iters, mh, "dense", docs, ragged and not refresh, K, V, lam, T, 0,
                     refresh, not refresh and rng.random() < 0.3, 0, rng.choice((0, 0, iters)))
    if family in ("mixture", "steps"):
        K = spread(50, min(16_000, 1.4e9 / V))
        mh = rng.choice((5, 6, 8)) if family == "steps" else mh
        return _case("", base, min(iters, 3) if family == "steps" else iters, mh, "mixture", docs,
                     ragged, K, V, lam, T, loglik_every=rng.choice((0, 0, iters)))
    if family == "hybrid":
        K = spread(13_000, 150_000)
        V = spread(30_000, 600_000)
        rows = spread(100, min(V // 2, 1e9 / K))
        return _case("", "c4", min(iters, 3), 2, "hybrid", docs, ragged, K, V, lam, 0, rows)
    K = spread(50_000, 1_000_000)
    block = max(20_000, int(docs * lam / rng.uniform(2.0, 6.0))) if family == "streamed" else 0
    return _case("", "c5", min(iters, 3), 2, "hybrid", docs, ragged, K, V, lam, 0, -1, block=block)


def _corpus(case, seed):
    # every seed gives exactly D * lam tokens: some more documents are made and the rest cut off
    D, n = case["D"], int(case["D"] * case["lam"])
    cfg = replace(corpus.CONFIGS["c1"], D=D + 2 + int(8.0 * math.sqrt(D / case["lam"])),
                  lam=case["lam"], V=case["V"], s=case["s"], T=case["T"], gen_seed=seed)
    doff, words = corpus.make_corpus(cfg)
    doff = np.append(doff[: np.searchsorted(doff, n)], n)
    words = np.ascontiguousarray(words[:n])
    if case["ragged"]:
        # the same tokens cut into documents of log-normal lengths, one in fifty of them empty
        rng = np.random.default_rng(seed)
        cut = np.exp(rng.normal(0.0, 1.2, D)) * (rng.random(D) > 0.02)
        doff = np.concatenate([[0], np.floor(np.cumsum(cut) / cut.sum() * n)]).astype(np.int64)
        doff[-1] = n
    return doff, words


class _Job:
    """A training program: the sampler, its stream, and the buffer it checkpoints z into."""


def prepare(case, seed):
    doff, words = _corpus(case, seed)
    opts = {}
    if case["store"] == "mixture":
        opts["dense_alias_min_count"] = case["K"]
    elif case["store"] == "hybrid":
        # dense tables only for words that have a dense row and at least K tokens
        tail = np.bincount(words, minlength=case["V"])[max(case["dense_rows"], 0):]
        opts.update(dense_rows=case["dense_rows"],
                    dense_alias_min_count=max(int(tail.max()) + 1, case["K"]))
    job = _Job()
    job.case = case
    job.stream = torch.cuda.Stream()
    job.model = lda.Lda(doff, words, case["V"], case["K"], case["alpha"], case["beta"], seed=seed,
                        stream=job.stream.cuda_stream, doc_refresh=int(case["refresh"]),
                        stream_block_tokens=case["block"], **opts)
    job.z = torch.empty(job.model.N, dtype=torch.int32, pin_memory=True).numpy()
    return job


def run(job):
    m, case = job.model, job.case
    out = {"loglik": []}
    for it in range(case["iters"]):
        m.build_alias()
        m.sweep(case["mh"])
        if case["update"]:
            m.update_counts()
        else:
            m.rebuild_counts()
        if case["loglik_every"] and (it + 1) % case["loglik_every"] == 0:
            out["loglik"].append(m.loglik())
    # lda_get_z itself, for the program's own pinned buffer (Lda.get_z allocates one)
    m._ck(lda.load_library().lda_get_z(m._h, job.z))
    out["z"] = job.z
    out["nk"] = m.get_nk()
    return out


def work(case):
    """Per iteration: a token's word and topic read, its new topic written; per count or table
    entry the count read, a bin of 8 bytes and the new count written.  A word of the mixture
    form has no more entries than tokens.  Then the assignment copied out."""
    n = case["D"] * case["lam"]
    V, K = case["V"], case["K"]
    p = np.arange(1, V + 1, dtype=np.float64) ** -case["s"]
    count = n * p / p.sum()
    if case["store"] == "dense":
        entries = float(V) * K
    else:
        entries = float(np.minimum(count, K).sum())
    looks = case["iters"] // case["loglik_every"] if case["loglik_every"] else 0
    return {"bytes": case["iters"] * (12.0 * n + 16.0 * entries) + looks * (4.0 * n + 4.0 * entries) + 4.0 * n,
            # two products of four factors and the comparison, per step
            "flops": case["iters"] * case["mh"] * n * 12.0}


def tolerance(case):
    """Assignments and counts are whole numbers and stay the same.  The log-likelihood is a sum of
    10^5 to 10^8 lgamma values in fp64: 1.5e-16 from an exactly rounded sum of the same terms at
    2 * 10^6 tokens; a tree of 27 levels of roundings bounds it at about 3e-15."""
    return {"rel": 1e-14, "max": 1e-14, "differ": 0.0} if case["loglik_every"] else "exact"
