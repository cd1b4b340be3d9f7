"""The work a user of this library has it do, as cases that can be timed: training passes on
corpora from a few thousand tokens to the size of the largest benchmark workload, and the
exchange of a saved state.

A case names a corpus (documents, vocabulary, length law), the number of topics, how the corpus is
held on the GPU and what one pass does:

  "train"     `iters` iterations in one call, then the log-likelihood and the new assignments are
              fetched: a stretch of training between two checkpoints.  With `loglik` every
              iteration evaluates the likelihood of its state (as bench.py does), without it the
              likelihood is evaluated once at the end (as the training loop of bow.py does).
  "exchange"  a saved state is installed, scored, and the model is taken out: the document-topic
              rows, the word-topic matrix, the topic totals.

A context keeps its state between passes, so a repeated training pass continues the chain.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import corpus_synth
import paper_1803_04631_amd as mlda


def _named(name, config, **more):
    """A case on the corpus shape of one of the benchmark's configurations."""
    c = corpus_synth.CONFIGS[config]
    case = {"name": name, "do": "train", "D": c.D, "V": c.V, "K": c.K, "law": c.length_law,
            "mean_len": c.mean_len, "sigma": c.sigma, "zipf_s": c.zipf_s, "alpha_gen": c.alpha_gen,
            "start": "random", "iters": 1, "loglik": False, "chunks": 1}
    case.update(more)
    return case


def _free(name, D, V, K, mean_len, law="poisson", sigma=0.0, **more):
    case = {"name": name, "do": "train", "D": D, "V": V, "K": K, "law": law, "mean_len": float(mean_len),
            "sigma": sigma, "zipf_s": 1.1, "alpha_gen": 0.1, "start": "random", "iters": 1,
            "loglik": False, "chunks": 1}
    case.update(more)
    return case


def listed():
    return [
        # The smallest call: one iteration on the corpus of the smoke check (8,000 tokens), where
        # launches and the calls' own cost are everything.
        _free("tiny", 200, 300, 24, 40, loglik=True),
        # The small configurations with their own numbers of topics: a corpus one would try
        # parameters on; a thousand documents, then twenty thousand.
        _named("small", "C1", iters=10, loglik=True),
        _named("medium", "C2", iters=5),
        # News articles (the benchmark's shape of the paper's first corpus), late in training: the
        # rows of theta are those of the topics the corpus was generated with.
        _named("news_late", "C3", start="generated", iters=5),
        # Abstracts (the shape of the paper's second corpus), the benchmark's default workload and the
        # largest: the likelihood is evaluated every iteration, from random topics.
        _named("abstracts", "C4", iters=10, loglik=True),
        # The upper end of the paper's range of K on the news corpus.
        _named("news_ten_thousand_topics", "C5", iters=3),
        # An odd K between the two: 4-byte rows, workgroups of four waves; ragged sizes everywhere.
        _free("mid_topics", 30011, 25013, 1537, 211, "lognormal", 0.6, iters=5),
        # Books: few, very long documents over few topics, counts far beyond one entry of a row.
        _free("books", 311, 40009, 299, 30000, "lognormal", 0.7, iters=3),
        # More topics than the on-chip column of a word's weights has room for.
        _free("forty_thousand_topics", 8009, 6007, 40000, 250, iters=2),
        # The news corpus in four chunks that take turns on the GPU: what a corpus larger than
        # the device's memory does.
        _named("news_streamed", "C3", iters=2, loglik=True, chunks=4),
        # A saved state of a fifth of the news corpus installed, scored and exported.
        _named("exchange", "C3", D=60000, do="exchange", start="generated"),
    ]


def draw(rng):
    """Any size of the listed range: tokens, vocabulary, topics and document lengths are spread over
    their logarithms and come out ragged."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    K = log_int(8, 60000)
    tokens = log_int(6000, min(3.0e8, 1.2e12 / max(K, 4000)))
    V = log_int(60, min(140000, 1.0e9 / K, tokens / 10))
    mean_len = log_int(8, min(30000, tokens / 4))
    law = rng.choice(["poisson", "lognormal"])
    kind = rng.choice(["train", "train", "train", "train", "streamed", "exchange"])
    case = {"do": "train", "D": max(2, int(tokens / mean_len)), "V": V, "K": K, "law": law,
            "mean_len": float(mean_len), "sigma": round(rng.uniform(0.2, 0.7), 2) if law == "lognormal" else 0.0,
            "zipf_s": round(rng.uniform(1.0, 1.2), 2), "alpha_gen": rng.choice([0.05, 0.1]),
            "start": rng.choice(["random", "generated"]), "iters": rng.randint(1, 5),
            "loglik": rng.random() < 0.5, "chunks": 1}
    if kind == "streamed":
        case["chunks"] = rng.randint(2, 6)
    if kind == "exchange" and V * K <= 1.2e8 and tokens <= 3e7:
        case.update(do="exchange", start="generated", iters=1, loglik=False)
    return case


@functools.lru_cache(maxsize=1)
def _corpus(D, V, K, law, mean_len, sigma, zipf_s, alpha_gen):
    return corpus_synth.generate(corpus_synth.CorpusConfig("case", D, V, K, law, mean_len, sigma, zipf_s,
                                                           alpha_gen, 0.01, 1))


def prepare(case, seed):
    """The corpus on the GPU in a context that has its start state, as a training program holds it.
    The case fixes the corpus up to its numbering (so that every seed gives arrays of the same sizes);
    the seed numbers the words, the documents and the topics and keys the library's generator."""
    D, V, K = case["D"], case["V"], case["K"]
    corpus = _corpus(D, V, K, case["law"], case["mean_len"], case["sigma"], case["zipf_s"], case["alpha_gen"])
    gen = torch.Generator().manual_seed(seed)
    first = int(torch.randint(D, (1,), generator=gen))                  # the document that comes first
    word_number = torch.randperm(V, generator=gen).to(torch.int32)
    topic_number = torch.randperm(K, generator=gen).to(torch.int32).numpy().astype(np.uint16)
    cut = int(corpus.doc_ptr[first])
    doc_ptr = np.concatenate([corpus.doc_ptr[first:] - cut, corpus.doc_ptr[1:first + 1] + (corpus.T - cut)])
    old_ids = torch.from_numpy(corpus.word_ids)
    word_ids = torch.cat([word_number[old_ids[cut:]], word_number[old_ids[:cut]]]).numpy()
    model = mlda.Mlda(doc_ptr, word_ids, V, K, 50.0 / K, 0.01, seed, chunks=case["chunks"])
    state = {"case": case, "model": model}
    if case["start"] == "random":
        model.init_random()
        return state
    z = topic_number[np.concatenate([corpus.z_true[cut:], corpus.z_true[:cut]])]
    if case["do"] == "exchange":
        state["z"] = z
    else:
        model.set_assignments(z)
    return state


def run(state):
    case, model = state["case"], state["model"]
    if case["do"] == "exchange":
        model.set_assignments(state["z"])
        loglik = model.loglik()
        row_ptr, topics, counts = model.doc_topic_csr()
        return {"loglik": loglik, "row_ptr": row_ptr, "topics": topics, "counts": counts,
                "word_topic": model.word_topic(), "topic_totals": model.topic_totals()}
    model.step(case["iters"], loglik=case["loglik"])
    return {"loglik": model.loglik(), "assignments": model.assignments(), "topic_totals": model.topic_totals()}


def _expected(case):
    """Tokens and expected non-zero entries of theta: per document, and per token's document."""
    n, K = case["mean_len"], case["K"]
    biased = n * math.exp(case["sigma"] ** 2) if case["law"] == "lognormal" else n + 1.0
    # (topics of a document spread evenly over all K: an upper bound that a random start reaches)
    entries = lambda length: K * -math.expm1(-length / K)       # noqa: E731
    return case["D"] * n, entries(n), entries(biased)


def work(case):
    """One pass: per iteration every token's word, document, old and new topic, both matrices of
    counts read once and written once (2-byte cells), and for every token a multiplication and
    an addition per entry of its document's row."""
    T, per_doc, per_token = _expected(case)
    D, V, K = case["D"], case["V"], case["K"]
    entry = 2 if K < 1024 else 4
    phi, theta = 2.0 * V * K, entry * D * per_doc
    if case["do"] == "exchange":        # the state in; the rows, the matrix and the totals out
        return {"bytes": 2 * T + 8 * D + 6 * D * per_doc + 4.0 * V * K + 4 * K, "flops": 0.0}
    once = 12 * T + 2 * phi + 2 * theta
    return {"bytes": case["iters"] * once + 2 * T, "flops": case["iters"] * 2 * T * per_token}


def tolerance(case):
    """Counts and assignments are whole numbers.  A draw falls on the other side of a prefix sum only
    where two orders of summation in fp64 round differently: the bar of the parity tests, 1e-6 of the
    tokens, though none has been seen.  The likelihood is an fp64 sum of up to 1e9 terms (4e-13 seen
    between orders)."""
    return {"rel": 2e-12, "differ": 1e-6}
