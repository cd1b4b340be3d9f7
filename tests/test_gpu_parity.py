"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle on the
same seeded inputs.  Bars: integer work (initial topics, counts, CSR rows) bit-exact;
sampled assignments may differ from the oracle on at most 1e-6 of the tokens (fp64
rounding order at a CDF boundary); log-likelihood within 1e-5 relative."""
import ctypes

import numpy as np
import pytest

import corpus_synth
import oracle

pytestmark = pytest.mark.gpu

Z_MISMATCH_FRACTION = 1e-6
LL_RTOL = 1e-5
SEED = corpus_synth.SAMPLER_SEED


@pytest.fixture(scope="module")
def mlda():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible: the gpu-marked tests need a real MI355X")
    import paper_1803_04631_amd as m
    m.load_library()
    return m


def say(*a):
    print(*a, flush=True)


def check_counts(model, c, z, V, K):
    """Counts held by the library == a recount of z by the oracle (bit-exact)."""
    n_wk, n_k = oracle.count_word_topic(c.word_ids, z, V, K)
    assert np.array_equal(model.word_topic(), n_wk)
    assert np.array_equal(model.topic_totals(), n_k)
    row_ptr, topics, counts = oracle.doc_topic_csr(c.doc_ptr, z, K)
    g_ptr, g_top, g_cnt = model.doc_topic_csr()
    assert np.array_equal(g_ptr, row_ptr)
    assert np.array_equal(g_top, topics)
    assert np.array_equal(g_cnt, counts)
    assert model.doc_topic_nnz() == row_ptr[-1]
    assert n_wk.sum() == counts.sum() == len(z) and n_k.sum() == len(z)
    return n_wk, n_k


def check_step(model, c, z, V, K, alpha, beta, seed, it):
    """One iteration from state z on both sides; returns the GPU's new state."""
    n_wk, n_k = oracle.count_word_topic(c.word_ids, z, V, K)
    want = oracle.iteration(c.doc_ptr, c.word_ids, z, V, K, alpha, beta, seed, it, n_wk, n_k)
    model.step(1)
    got = model.assignments()
    assert got.max(initial=0) < K
    bad = int((got != want).sum())
    assert bad <= Z_MISMATCH_FRACTION * len(z), f"{bad} of {len(z)} assignments differ at iteration {it}"
    n_wk2, n_k2 = check_counts(model, c, got, V, K)
    ll = oracle.loglik(c.doc_ptr, got, V, K, alpha, beta, n_wk2, n_k2)
    assert abs(model.loglik() - ll) <= LL_RTOL * abs(ll)
    return got


def test_philox_bitwise(mlda):
    n = 1 << 20
    for seed, it, t0 in [(SEED, 1, 0), (2**63 + 12345, 77, 2**32 - 1000), (0, 0, 2**40)]:
        say("philox", seed, it, t0)
        got = mlda.philox_uniform(seed, it, t0, n).cpu().numpy()
        assert np.array_equal(got, oracle.uniforms(seed, it, t0, n))


@pytest.mark.parametrize("name,iters", [("C1", 10), ("C2", 6)])
def test_named_config_free_running(mlda, name, iters):
    """Configs C1 and C2: initial state, then every iteration, against the oracle."""
    c = corpus_synth.generate(name)
    cfg = c.config
    say(name, "T", c.T)
    model = mlda.Mlda(c.doc_ptr, c.word_ids, cfg.V, cfg.K, cfg.alpha, cfg.beta, SEED)
    model.init_random()
    z = oracle.init_topics(c.T, cfg.K, SEED)
    assert np.array_equal(model.assignments(), z)
    check_counts(model, c, z, cfg.V, cfg.K)
    nnz = [model.doc_topic_nnz()]
    for it in range(1, iters + 1):
        say(name, "iteration", it)
        z = check_step(model, c, z, cfg.V, cfg.K, cfg.alpha, cfg.beta, SEED, it)
        nnz.append(model.doc_topic_nnz())
        assert model.iteration == it
    assert nnz[-1] < nnz[0]          # Section 7.1: theta gets sparser over the first iterations
    model.close()


def test_converged_like_state(mlda):
    """Start from the topics the corpus was generated with (sparse theta rows)."""
    c = corpus_synth.generate("C2")
    cfg = c.config
    model = mlda.Mlda(c.doc_ptr, c.word_ids, cfg.V, cfg.K, cfg.alpha, cfg.beta, SEED)
    model.set_assignments(c.z_true, it=40)
    assert model.iteration == 40
    assert np.array_equal(model.assignments(), c.z_true)
    check_counts(model, c, c.z_true, cfg.V, cfg.K)
    check_step(model, c, c.z_true, cfg.V, cfg.K, cfg.alpha, cfg.beta, SEED, 41)
    model.close()


EDGE_CASES = [
    # name,                 D,   V,    K,   mean_len
    ("single_topic",        50,  30,   1,   10),
    ("two_topics",          50,  30,   2,   10),
    ("k_not_mult_of_16",    80,  60,   37,  30),
    ("k_just_over_wave",    60,  90,   65,  300),     # rows longer than one wave
    ("long_rows",           40,  500,  300, 2500),    # nnz up to ~300: several row chunks
    ("one_word_vocab",      40,  1,    8,   20),
    ("large_k_small_docs",  300, 2000, 10000, 120),   # C5-like K: 45 KB of LDS per tile
    ("short_docs",          3000, 200, 16,  1.2),     # many single-token documents (S = 0)
    # large K, words of every size: several tiles, one tile of more than 1024 tokens, and
    # small ones, which one workgroup takes in runs of 16 (p* of a word derived from the word before)
    ("large_k_mixed_words", 400, 70,   3000, 300),
    ("k_twenty_thousand",   40,  300,  20000, 400),   # every kernel beyond 64 KB of LDS
    ("k_near_lds_limit",    40,  300,  30800, 400),   # 160 KB of LDS: one workgroup per CU
    # K whose p* does not fit a workgroup's LDS: p* of a tile in device memory, a fixed number of
    # workgroups that take tile after tile (1,500 words: more tiles than workgroups); beyond
    # 32,768 topics the histograms of phi and n_k are taken in two ranges of topics
    ("k_beyond_lds",         40,  300,  31000, 400),
    ("k_beyond_lds_many_words", 200, 1500, 33000, 40),
    ("k_largest",            30,  200,  65535, 300),
    # long documents over few topics: counts up to 1,000 in 4-byte entries
    ("huge_docs_split_rows", 3,   400,  700, 17000),
    ("huge_docs_few_topics", 4,   50,   24,  16500),
    # rows too long for the kept pass shapes: walked twice by a whole wave
    ("rows_over_768",        6,   300,  1200, 9000),
    ("rows_over_768_split",  3,   300,  1100, 17500),
    ("rows_near_k_1023",     3,   300,  1023, 30000),
    # 2-byte entries with six bits of count up to K = 1,023, five up to 2,047, three at 2,048
    ("k_last_six_bits",      30,  300,  1023, 600),
    ("k_first_five_bits",    30,  300,  1024, 400),
    ("k_last_five_bits",     30,  300,  2047, 600),
    ("k_2048_three_bits",    30,  300,  2048, 600),
]


# Where the layouts of a theta row meet: (name, D, V, K, mean length).  Up to K = 2048 a row has 2-byte
# entries with three bits of count (short documents), six (K < 1024) or five (K < 2048), or, for documents
# long beside the topics, 4-byte entries with counts up to 8,191; beyond, 4-byte entries with 16,383.
LAYOUT_CASES = [
    ("counted_few_topics",     60, 80,   24,   55),
    ("six_bits_wider_rows",    25, 120,  200,  700),    # eight and more lanes to a row
    ("counted_from_here",      60, 80,   24,   110),
    ("counted_splits",         2,  60,   2,    30000),  # counts beyond 8,191
    ("counted_wide_counters",  2,  60,   5,    70000),  # 2^16 tokens in a document
    ("counts_beyond_16_bits",  2,  40,   1,    70000),
    ("five_bits_long_docs",    3,  300,  2000, 5000),   # sixteen waves count a document; beyond the widest shape
    ("packed_long_docs",       3,  300,  3000, 5000),
    ("k_one",                  20, 30,   1,    40),
    ("k_largest_fp64",         25, 200,  2048, 300),
    ("k_first_fp32",           25, 200,  2049, 300),
    ("counted_longest_rows",   4,  300,  2048, 2500),   # beyond the widest pass shape
    # 4-byte entries and fp32 weights again, workgroups of four waves: the shortest documents ...
    ("packed_four_waves",      300, 50,  1024, 30),
    ("packed_four_waves_2048", 300, 50,  2048, 30),
    ("three_bits_from_here",   60, 50,   2048, 260),
    # ... and words of few tokens
    ("packed_small_words",     60, 3000, 1500, 150),
]


@pytest.mark.parametrize("wide_offsets", ["0", "1"])
@pytest.mark.parametrize("case", LAYOUT_CASES, ids=[c[0] for c in LAYOUT_CASES])
def test_row_layouts(mlda, case, wide_offsets, monkeypatch):
    monkeypatch.setenv("MLDA_WIDE_SLOT_OFFSETS", wide_offsets)
    name, D, V, K, mean_len = case
    c = corpus_synth.tiny(D=D, V=V, K=K, mean_len=mean_len, seed=len(name), name=name)
    alpha, beta = 50.0 / K, 0.01
    say(name, "T", c.T)
    model = mlda.Mlda(c.doc_ptr, c.word_ids, V, K, alpha, beta, SEED)
    model.init_random()
    z = oracle.init_topics(c.T, K, SEED)
    assert np.array_equal(model.assignments(), z)
    for it in (1, 2, 3):
        z = check_step(model, c, z, V, K, alpha, beta, SEED, it)
    model.close()


# (name, K, document lengths as (how many, tokens))
SPLIT_CASES = [
    ("three_bits",               1000, [(60, 300)]),
    ("three_bits_pair_of_docs",  120,  [(200, 140)]),
    ("five_bits",                1500, [(20, 1500)]),
    ("six_bits",                 500,  [(20, 1500)]),
    ("six_bits_pair_of_docs",    60,   [(200, 150)]),
    ("six_bits_sixteen_waves",   1000, [(6, 5000)]),
    ("six_bits_wide_counters",   1023, [(100, 4000), (1, 66000)]),
    ("counted",                  24,   [(40, 600)]),
    ("counted_sixteen_waves",    24,   [(4, 30000)]),
    ("packed",                   3000, [(6, 40000)]),
]


@pytest.mark.parametrize("wide_offsets", ["0", "1"])
@pytest.mark.parametrize("case", SPLIT_CASES, ids=[c[0] for c in SPLIT_CASES])
def test_counts_at_the_ends_of_their_fields(mlda, case, wide_offsets, monkeypatch):
    """Counts of exactly what an entry of each layout holds and one more (7, 15, 31, 63, 8,191, 16,383
    and their doubles, as far as the document goes), the rest of the document in its first, a middle
    and its last topic, so that a topic's entries run across units and lanes; beside documents
    spread over all topics (rows beyond the widest shape where K is large)."""
    monkeypatch.setenv("MLDA_WIDE_SLOT_OFFSETS", wide_offsets)
    name, K, docs = case
    V, alpha, beta = 60, 50.0 / K, 0.01
    lens = np.concatenate([np.full(n, length, dtype=np.int64) for n, length in docs])

    class C:  # minimal corpus record
        pass
    c = C(); c.doc_ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64); c.T = int(lens.sum())
    rng = np.random.default_rng(len(name))
    c.word_ids = rng.integers(V, size=c.T).astype(np.int32)
    z = rng.integers(K, size=c.T).astype(np.uint16)
    for d, n in enumerate(lens):
        if d % 2:
            continue
        row = np.empty(n, dtype=np.uint16)
        at = 0
        for k, count in enumerate([7, 8, 14, 15, 16, 31, 32, 63, 64, 126, 127, 8191, 8192, 16383, 16384]):
            if at + count <= n // 2 or (count > 8000 and at + count <= n):
                row[at:at + count] = 1 + k
                at += count
        row[at:] = rng.choice([0, K // 2, K - 1], size=n - at)
        z[c.doc_ptr[d]:c.doc_ptr[d + 1]] = rng.permutation(row)
    model = mlda.Mlda(c.doc_ptr, c.word_ids, V, K, alpha, beta, SEED)
    model.set_assignments(z)
    check_counts(model, c, z, V, K)
    for it in (1, 2):
        z = check_step(model, c, z, V, K, alpha, beta, SEED, it)
    model.close()


# (MLDA_TILE_SHAPE: tokens of a tile, and up to how many of them one wave takes a tile alone)
@pytest.mark.parametrize("shape", ["1024,0", "128,128", "256,40"])
@pytest.mark.parametrize("case", [c for c in LAYOUT_CASES if c[3] <= 2048], ids=lambda c: c[0])
def test_row_layouts_in_every_tile_shape(mlda, case, shape, monkeypatch):
    """Workgroups of four waves, of one, and both side by side, on corpora that would take another shape."""
    monkeypatch.setenv("MLDA_TILE_SHAPE", shape)
    test_row_layouts(mlda, case, "1" if shape == "128,128" else "0", monkeypatch)


@pytest.mark.parametrize("case", [c for c in SPLIT_CASES if c[1] <= 2048], ids=lambda c: c[0])
def test_counts_at_the_ends_of_their_fields_with_four_waves(mlda, case, monkeypatch):
    monkeypatch.setenv("MLDA_TILE_SHAPE", "1024,0")
    test_counts_at_the_ends_of_their_fields(mlda, case, "0", monkeypatch)


@pytest.mark.parametrize("chunks", [1, 3])
def test_tile_shapes_agree(mlda, chunks, monkeypatch):
    """Words of 1 .. 2,100 tokens (tiles of every size), the same assignments and byte counts in every shape."""
    V, K = 120, 200
    rng = np.random.default_rng(3)
    per_word = np.concatenate([np.arange(1, 100), [127, 128, 129, 255, 256, 257, 1023, 1024, 1025, 2100], np.zeros(11, int)])
    words = rng.permutation(np.repeat(np.arange(V, dtype=np.int32), per_word))
    doc_ptr = np.concatenate([[0], np.sort(rng.choice(np.arange(1, len(words)), 150, replace=False)), [len(words)]]).astype(np.int64)
    got = []
    for shape in ("1024,0", "64,64", "128,128", "256,64", "1024,64", ""):
        monkeypatch.setenv("MLDA_TILE_SHAPE", shape)
        model = mlda.Mlda(doc_ptr, words, V, K, 50.0 / K, 0.01, SEED, chunks=chunks)
        model.init_random(); model.step(3)
        got.append((model.assignments(), model.sampler_bytes(), model.loglik()))
        model.close()
    for z, moved, ll in got[1:]:
        assert np.array_equal(z, got[0][0]) and np.array_equal(moved, got[0][1]) and ll == got[0][2]



# Rows of every way the walk over fp64 weights goes: (name, K, documents, tokens each).
SMALL_BETA_CASES = [
    ("two_byte_rows",         60,   400, 50),
    ("two_byte_rows_wider",   300,  60,  400),
    ("two_byte_rows_six_bits", 300, 20,  1000),
    ("two_byte_longest_rows", 2000, 3,   5000),
    ("four_byte_rows",        24,   40,  600),
    ("four_byte_longest_rows", 2000, 2,  17000),
]


@pytest.mark.parametrize("beta", [1e-10, 1e-14, 1e-30])
@pytest.mark.parametrize("case", SMALL_BETA_CASES, ids=[c[0] for c in SMALL_BETA_CASES])
def test_small_beta(mlda, case, beta):
    """Words seen once or twice under a beta far below 1: p* of the token's own topic is 1/beta
    times what is left of it without the token, and than the other topics'.  A sum that held it and
    gave it back would have nothing left of the rest; alpha is so small that the row decides.
    (p* stays a normal fp32 number: beta / n_k > 1e-36.)"""
    name, K, D, length = case
    T, V = D * length, D * length // 2
    rng = np.random.default_rng(K + D)

    class C:  # minimal corpus record
        pass
    c = C(); c.doc_ptr = np.arange(D + 1, dtype=np.int64) * length; c.T = T
    c.word_ids = rng.integers(V, size=T).astype(np.int32)
    alpha = 1e-30
    model = mlda.Mlda(c.doc_ptr, c.word_ids, V, K, alpha, beta, SEED)
    model.init_random()
    z = oracle.init_topics(T, K, SEED)
    for it in (1, 2):
        z = check_step(model, c, z, V, K, alpha, beta, SEED, it)
    model.close()


# (topics, tokens of a document, documents, words): many tokens of a document share a word, so their rows are walked
# once.  Rows of every pass shape: up to 4, 8, 12 units of a row on 4 lanes, 16, 24 on 8, 32, 48 on 16, 64, 96 on
# 32, 128, 192 on 64 (2-byte entries: 8 to a unit), and longer ones, which are not shared.
SHARED_CASES = [(2000, n, D, 4) for n, D in [(60, 300), (90, 250), (125, 200), (185, 150), (250, 100), (370, 70),
                                             (500, 50), (780, 40), (1200, 30), (2000, 20), (4000, 8)]] + [
    # a sum per sub-lane, 4 entries to a unit; rows beyond the widest shape; counts of several entries; p* in device memory
    (2500, 100, 200, 3), (2500, 130, 150, 3), (2500, 200, 100, 3), (2500, 300, 80, 3), (2500, 400, 60, 3), (2500, 700, 40, 3),
    (2500, 1100, 30, 3), (2500, 3000, 12, 3), (3000, 40000, 4, 3), (40000, 300, 30, 3), (40000, 3000, 6, 3), (65535, 150, 40, 2),
    (24, 200, 150, 4), (24, 30, 400, 2), (300, 28, 600, 2), (300, 500, 40, 5), (1023, 700, 30, 5), (1, 64, 40, 2)]


@pytest.mark.parametrize("shape", ["1024,0", "128,128"])
@pytest.mark.parametrize("case", SHARED_CASES, ids=lambda c: "k%d_n%d" % c[:2])
def test_walks_shared_by_tokens(mlda, case, shape, monkeypatch):
    monkeypatch.setenv("MLDA_TILE_SHAPE", shape)
    monkeypatch.setenv("MLDA_WIDE_SLOT_OFFSETS", "1" if shape == "128,128" else "0")
    K, length, D, V = case
    rng = np.random.default_rng(K + length)
    lens = np.maximum(1, length + rng.integers(-3, 4, size=D))

    class C:  # minimal corpus record
        pass
    c = C(); c.doc_ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64); c.T = int(lens.sum())
    c.word_ids = rng.integers(V, size=c.T).astype(np.int32)
    spread = rng.integers(K, size=c.T).astype(np.uint16)
    # topics whose counts take many entries, which then cross units and lanes
    few = np.where(rng.random(c.T) < 0.8, rng.choice([0, K // 3, K // 2, K - 1], size=c.T), spread).astype(np.uint16)
    model = mlda.Mlda(c.doc_ptr, c.word_ids, V, K, 50.0 / K, 0.01, SEED)
    for it, z in enumerate((spread, few)):
        model.set_assignments(z, it=it)
        check_step(model, c, z, V, K, 50.0 / K, 0.01, SEED, it + 1)
    model.close()


@pytest.mark.parametrize("K", [1, 11, 16, 17])
def test_few_topics_of_many_tokens(mlda, K):
    """Up to 16 topics of more than 10 million tokens: no walks are shared, though every document has its words many times."""
    D, length, V = 2501, 4000, 300
    rng = np.random.default_rng(K)

    class C:  # minimal corpus record
        pass
    c = C(); c.T = D * length; c.doc_ptr = np.arange(D + 1, dtype=np.int64) * length
    c.word_ids = rng.integers(V, size=c.T).astype(np.int32)
    z = ((c.word_ids * K // V + (rng.random(c.T) < 0.1) * rng.integers(K, size=c.T)) % K).astype(np.uint16)
    model = mlda.Mlda(c.doc_ptr, c.word_ids, V, K, 50.0 / K, 0.01, SEED)
    model.set_assignments(z)
    check_step(model, c, z, V, K, 50.0 / K, 0.01, SEED, 1)
    model.close()


@pytest.mark.parametrize("beta", [1e-3, 1e-5, 1e-9])
@pytest.mark.parametrize("case", [(2000, 4000, 8, 4), (300, 500, 40, 5), (24, 200, 150, 4), (299, 30000, 4, 40),
                                  (2500, 1100, 30, 3), (40000, 300, 30, 3)], ids=lambda c: "k%d_n%d" % c[:2])
def test_walks_shared_where_sums_round(mlda, case, beta):
    """Some topics hold most tokens of some words and none of others: of the rows' sums some are exact, some too long by a
    bit or two, and some by many (those tokens' walks are their own)."""
    K, length, D, V = case
    rng = np.random.default_rng(K)

    class C:  # minimal corpus record
        pass
    c = C(); c.T = D * length; c.doc_ptr = np.arange(D + 1, dtype=np.int64) * length
    c.word_ids = rng.integers(V, size=c.T).astype(np.int32)
    group = (c.word_ids.astype(np.int64) * K // V + rng.integers(max(1, K // V), size=c.T)) % K       # topics of the word's own
    z = np.where(rng.random(c.T) < 0.9, group, rng.integers(K, size=c.T)).astype(np.uint16)
    model = mlda.Mlda(c.doc_ptr, c.word_ids, V, K, 50.0 / K, beta, SEED)
    model.set_assignments(z)
    for it in (1, 2):
        z = check_step(model, c, z, V, K, 50.0 / K, beta, SEED, it)
    model.close()


@pytest.mark.parametrize("beta", [0.01, 1e-14, 1e-30])
@pytest.mark.parametrize("K", [30, 500, 3000, 31000])
def test_shared_walks_with_little_left(mlda, K, beta):
    """Documents with one token of a word, its only one of its topic, among documents of that word alone: without the
    token nothing of the row's sum is left but beta, and alpha is too small to matter.  (Documents of fewer than 90 tokens
    do not share walks beyond K = 2,048; K = 31,000 has its weights in device memory.)"""
    V, pairs, length = 3, 11, 40 if K <= 2048 else 100
    half = length // 2
    words, z = [], []
    for i in range(pairs):
        words += [0] * length + [0] + [1] * (length - 1)
        z += [0] * length + [2 + i] + [K - 1] * half + [K - 2] * (length - 1 - half)

    class C:  # minimal corpus record
        pass
    c = C(); c.doc_ptr = np.arange(2 * pairs + 1, dtype=np.int64) * length; c.T = 2 * length * pairs
    c.word_ids = np.array(words, dtype=np.int32)
    z = np.array(z, dtype=np.uint16)
    model = mlda.Mlda(c.doc_ptr, c.word_ids, V, K, 1e-30, beta, SEED)
    for it in range(6):
        model.set_assignments(z, it=it)
        check_step(model, c, z, V, K, 1e-30, beta, SEED, it + 1)
    model.close()


@pytest.mark.parametrize("alpha", [1e-305, 1e-307])
@pytest.mark.parametrize("K", [16, 300])
def test_small_alpha(mlda, K, alpha):
    """Documents of one token, whose draw alpha alone decides, beside longer ones, under an alpha so
    small that alpha p* would be denormal with any factor to it."""
    D, V = 6000, 40
    rng = np.random.default_rng(K)
    lens = np.where(np.arange(D) % 4 == 0, 5, 1)

    class C:  # minimal corpus record
        pass
    c = C(); c.doc_ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64); c.T = int(lens.sum())
    c.word_ids = rng.integers(V, size=c.T).astype(np.int32)
    model = mlda.Mlda(c.doc_ptr, c.word_ids, V, K, alpha, 0.01, SEED)
    model.init_random()
    z = oracle.init_topics(c.T, K, SEED)
    for it in (1, 2):
        n_wk, n_k = oracle.count_word_topic(c.word_ids, z, V, K)
        want = oracle.iteration(c.doc_ptr, c.word_ids, z, V, K, alpha, 0.01, SEED, it, n_wk, n_k)
        model.step(1)
        z = model.assignments()
        assert np.array_equal(z, want)
    model.close()


@pytest.mark.parametrize("case", EDGE_CASES, ids=[c[0] for c in EDGE_CASES])
def test_edge_shapes(mlda, case):
    name, D, V, K, mean_len = case
    c = corpus_synth.tiny(D=D, V=V, K=K, mean_len=mean_len, seed=len(name), name=name)
    alpha, beta = 50.0 / K, 0.01
    say(name, "T", c.T)
    model = mlda.Mlda(c.doc_ptr, c.word_ids, V, K, alpha, beta, SEED)
    model.init_random()
    z = oracle.init_topics(c.T, K, SEED)
    assert np.array_equal(model.assignments(), z)
    for it in (1, 2, 3):
        z = check_step(model, c, z, V, K, alpha, beta, SEED, it)
    model.close()


@pytest.mark.parametrize("case", [("six_bits", 60, 90, 65, 300), ("five_bits", 30, 300, 1024, 600),
                                  ("counted_long_docs", 3, 300, 1100, 17500),
                                  ("large_k", 300, 2000, 10000, 120), ("k_beyond_lds", 40, 300, 31000, 400)],
                         ids=lambda c: c[0])
def test_wide_slot_offsets(mlda, case, monkeypatch):
    """The sampler kernels that address theta rows with 64-bit offsets (what rows beyond 4 GiB
    need; the full-size test of 2.1e9 tokens reaches only one of them), on small inputs."""
    name, D, V, K, mean_len = case
    monkeypatch.setenv("MLDA_WIDE_SLOT_OFFSETS", "1")
    c = corpus_synth.tiny(D=D, V=V, K=K, mean_len=mean_len, seed=len(name), name=name)
    alpha, beta = 50.0 / K, 0.01
    model = mlda.Mlda(c.doc_ptr, c.word_ids, V, K, alpha, beta, SEED)
    model.init_random()
    z = oracle.init_topics(c.T, K, SEED)
    for it in (1, 2):
        z = check_step(model, c, z, V, K, alpha, beta, SEED, it)
    model.close()


def test_long_document_with_more_topics_than_32bit_counters_fit(mlda):
    """A document of 2^16 tokens or more needs 32-bit counters in the theta rebuild; beyond
    32,768 topics they do not fit the LDS at once and the document is counted in two ranges of
    topics, its row growing range by range.  Counts beyond one entry's 16,383 in both ranges."""
    V, K = 50, 40000
    lens = np.array([70000, 300, 5, 0, 66000], dtype=np.int64)
    doc_ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    rng = np.random.default_rng(5)
    words = rng.integers(V, size=int(lens.sum())).astype(np.int32)
    z = rng.integers(K, size=len(words)).astype(np.uint16)
    z[0:20000] = 7                              # 20,000 tokens of a topic of the first range
    z[20000:38000] = 32767                      # the last topic of the first range
    z[38000:56000] = 32768                      # the first topic of the second
    z[56000:60000] = K - 1
    z[doc_ptr[4]:doc_ptr[4] + 40000] = 39000    # the last document: mostly one topic of the second range

    class C:  # minimal corpus record
        pass
    c = C(); c.doc_ptr = doc_ptr; c.word_ids = words; c.T = len(words)
    alpha, beta = 50.0 / K, 0.01
    model = mlda.Mlda(doc_ptr, words, V, K, alpha, beta, SEED)
    model.set_assignments(z, it=0)
    assert np.array_equal(model.assignments(), z)
    check_counts(model, c, z, V, K)
    check_step(model, c, z, V, K, alpha, beta, SEED, 1)
    model.close()


@pytest.mark.parametrize("K", [500, 1500])
def test_counts_beyond_one_entry(mlda, K):
    """Documents whose tokens sit in one or two topics: counts of 20,000 to 70,000, which no entry
    of a theta row holds (8,191 at most),
    so that a topic takes several entries in a row, also across the lanes of the row walk; a
    document of 2^16 tokens or more needs 32-bit counters in the rebuild."""
    V = 60
    lens = np.array([70000, 40000, 20000, 300, 17, 1, 16384, 15, 16], dtype=np.int64)
    doc_ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    rng = np.random.default_rng(K)
    words = rng.integers(V, size=int(lens.sum())).astype(np.int32)
    z = rng.integers(K, size=len(words)).astype(np.uint16)
    z[doc_ptr[0]:doc_ptr[1]] = 3                                   # one topic
    z[doc_ptr[1]:doc_ptr[1] + 20000] = 0                           # two topics, at both ends of a row
    z[doc_ptr[1] + 20000:doc_ptr[2]] = K - 1
    z[doc_ptr[2]:doc_ptr[3]] = rng.integers(5, size=20000) * 7     # five topics
    z[doc_ptr[6]:doc_ptr[7]] = 11                                  # exactly 2^14 tokens of one topic
    z[doc_ptr[7]:doc_ptr[8]] = 2                                   # exactly 15
    z[doc_ptr[8]:doc_ptr[9]] = 2                                   # exactly 16

    class C:  # minimal corpus record
        pass
    c = C(); c.doc_ptr = doc_ptr; c.word_ids = words; c.T = len(words)
    alpha, beta = 50.0 / K, 0.01
    model = mlda.Mlda(doc_ptr, words, V, K, alpha, beta, SEED)
    model.set_assignments(z, it=0)
    assert np.array_equal(model.assignments(), z)
    check_counts(model, c, z, V, K)
    for it in (1, 2):
        z = check_step(model, c, z, V, K, alpha, beta, SEED, it)
    model.close()


# Rows whose slots are more than 512 KB and more than a byte per token, also of half the documents:
# (name, D, K, tokens each)
EXPORT_CASES = [
    ("three_bits", 7000, 100,  100),
    ("five_bits",  1000, 1500, 600),
    ("six_bits",   1040, 500,  600),
    ("counted",    10000,24,   110),
    ("packed",     1000, 3000, 300),
]


@pytest.mark.parametrize("chunks", [1, 2])
@pytest.mark.parametrize("case", EXPORT_CASES, ids=[c[0] for c in EXPORT_CASES])
def test_rows_laid_out_by_the_device(mlda, case, chunks):
    """The rows of theta are unpacked from a copy of small slots (the other tests) and laid out by the
    device otherwise, in every layout: spread rows beside rows of one topic of many entries."""
    name, D, K, length = case
    T, V = D * length, 50
    rng = np.random.default_rng(K)

    class C:  # minimal corpus record
        pass
    c = C(); c.doc_ptr = np.arange(D + 1, dtype=np.int64) * length; c.T = T
    c.word_ids = rng.integers(V, size=T).astype(np.int32)
    z = rng.integers(K, size=(D, length)).astype(np.uint16)
    z[::3] = rng.integers(K, size=(len(z[::3]), 1))
    z[1::3, length // 2:] = K - 1
    z = z.reshape(-1)
    model = mlda.Mlda(c.doc_ptr, c.word_ids, V, K, 0.1, 0.01, SEED, chunks=chunks)
    model.set_assignments(z)
    check_counts(model, c, z, V, K)
    model.close()


def test_mixed_row_lengths(mlda):
    """Documents of 3 to ~1500 tokens over few words: every group width and quad count of the
    row walk occurs, and the 64 tokens a wave takes together mix several of them."""
    V, K = 24, 2000
    parts = [corpus_synth.tiny(D=5, V=V, K=K, mean_len=m, seed=int(m), name="part")
             for m in (3, 12, 28, 45, 75, 110, 170, 300, 600, 1000, 1500)]
    lens = np.concatenate([np.diff(p.doc_ptr) for p in parts])
    order = np.random.default_rng(5).permutation(len(lens))          # lengths in no order
    starts = np.concatenate([[0], np.cumsum(lens)])
    words_by_doc = np.concatenate([p.word_ids for p in parts])
    words = np.concatenate([words_by_doc[starts[d]:starts[d + 1]] for d in order]).astype(np.int32)
    doc_ptr = np.concatenate([[0], np.cumsum(lens[order])]).astype(np.int64)

    class C:  # minimal corpus record
        pass
    c = C(); c.doc_ptr = doc_ptr; c.word_ids = words; c.T = len(words)
    alpha, beta = 50.0 / K, 0.01
    say("mixed_row_lengths T", c.T, "longest", lens.max())
    model = mlda.Mlda(doc_ptr, words, V, K, alpha, beta, SEED)
    model.init_random()
    z = oracle.init_topics(c.T, K, SEED)
    nnz = np.diff(model.doc_topic_csr()[0])
    assert nnz.min() <= 16 and nnz.max() > 768      # from the narrowest shape to the widest
    for it in (1, 2, 3):
        z = check_step(model, c, z, V, K, alpha, beta, SEED, it)
    model.close()


def test_empty_documents_and_unused_words(mlda):
    base = corpus_synth.tiny(D=30, V=40, K=12, mean_len=9, seed=2)
    lens = np.diff(base.doc_ptr)
    # interleave empty documents, keep the same tokens; shift word ids so that word 0
    # and the last words never occur
    new_lens = np.zeros(2 * len(lens) + 3, dtype=np.int64)
    new_lens[1:2 * len(lens):2] = lens
    doc_ptr = np.concatenate([[0], np.cumsum(new_lens)]).astype(np.int64)
    words = (base.word_ids + 1).astype(np.int32)
    V, K, alpha, beta = 50, 12, 0.7, 0.05

    class C:  # minimal corpus record
        pass
    c = C(); c.doc_ptr = doc_ptr; c.word_ids = words; c.T = len(words)
    model = mlda.Mlda(doc_ptr, words, V, K, alpha, beta, 9)
    model.init_random()
    z = oracle.init_topics(c.T, K, 9)
    for it in (1, 2):
        z = check_step(model, c, z, V, K, alpha, beta, 9, it)
    n_wk = model.word_topic()
    assert n_wk[0].sum() == 0 and n_wk[41:].sum() == 0
    model.close()


@pytest.mark.parametrize("chunks", [2, 3, 7])
def test_streamed_chunks_match_oracle(mlda, chunks):
    """The corpus cut into chunks that take turns on the GPU (Algorithm 1, WorkSchedule2) gives
    the oracle's results like the resident corpus does."""
    c = corpus_synth.generate("C1")
    cfg = c.config
    model = mlda.Mlda(c.doc_ptr, c.word_ids, cfg.V, cfg.K, cfg.alpha, cfg.beta, SEED, chunks=chunks)
    model.init_random()
    z = oracle.init_topics(c.T, cfg.K, SEED)
    assert np.array_equal(model.assignments(), z)
    check_counts(model, c, z, cfg.V, cfg.K)
    for it in (1, 2, 3):
        say("streamed", chunks, "iteration", it)
        z = check_step(model, c, z, cfg.V, cfg.K, cfg.alpha, cfg.beta, SEED, it)
    # the log-likelihood evaluated inside the step, and two iterations in one call
    model.step(2, loglik=True)
    for it in (4, 5):
        n_wk, n_k = oracle.count_word_topic(c.word_ids, z, cfg.V, cfg.K)
        z = oracle.iteration(c.doc_ptr, c.word_ids, z, cfg.V, cfg.K, cfg.alpha, cfg.beta, SEED, it, n_wk, n_k)
    assert model.iteration == 5 and np.array_equal(model.assignments(), z)
    n_wk, n_k = check_counts(model, c, z, cfg.V, cfg.K)
    ll = oracle.loglik(c.doc_ptr, z, cfg.V, cfg.K, cfg.alpha, cfg.beta, n_wk, n_k)
    assert abs(model.loglik() - ll) <= LL_RTOL * abs(ll)
    ms, moved = model.timing(), model.sampler_bytes()      # per iteration, summed over the chunks
    assert ms.shape == (2, 4) and np.all(ms > 0) and moved.shape == (2,)
    assert np.all(moved >= 16.0 * c.T)
    model.close()


@pytest.mark.parametrize("chunks", [3, 4, 5, 8])
@pytest.mark.parametrize("order", ["long_first", "short_first", "long_and_empty"])
def test_streamed_chunks_of_different_shapes(mlda, order, chunks):
    """Chunks of few long documents and chunks of many short or empty ones take turns in the same two buffers, an odd number
    of them in the other one every iteration: one's records are copied in while another's assignments are copied out."""
    V, K, alpha, beta = 3000, 100, 0.5, 0.01
    lengths = np.repeat([300, 5], [1000, 60000])
    if order == "short_first":
        lengths = lengths[::-1]
    elif order == "long_and_empty":
        lengths = np.concatenate([np.full(1500, 200), np.zeros(150000, dtype=np.int64), np.full(1500, 200)])

    class C:
        pass
    c = C(); c.T = int(lengths.sum())
    c.doc_ptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    rng = np.random.default_rng(chunks)
    c.word_ids = np.minimum(rng.zipf(1.3, c.T) - 1, V - 1).astype(np.int32)
    say("different shapes", order, "chunks", chunks, "T", c.T)
    model = mlda.Mlda(c.doc_ptr, c.word_ids, V, K, alpha, beta, SEED, chunks=chunks)
    model.init_random()
    z = oracle.init_topics(c.T, K, SEED)
    assert np.array_equal(model.assignments(), z)
    for it in (1, 2, 3):
        z = check_step(model, c, z, V, K, alpha, beta, SEED, it)
    model.step(2, loglik=True)
    for it in (4, 5):
        n_wk, n_k = oracle.count_word_topic(c.word_ids, z, V, K)
        z = oracle.iteration(c.doc_ptr, c.word_ids, z, V, K, alpha, beta, SEED, it, n_wk, n_k)
    assert int((model.assignments() != z).sum()) <= Z_MISMATCH_FRACTION * c.T
    model.close()


def test_streamed_with_weights_in_device_memory(mlda):
    """K beyond the LDS column, the corpus in three chunks: p* in device memory, phi counted in
    two ranges of topics and added to chunk by chunk."""
    D, V, K = 30, 100, 33000
    c = corpus_synth.tiny(D=D, V=V, K=K, mean_len=100, seed=8, name="far_streamed")
    alpha, beta = 50.0 / K, 0.01
    model = mlda.Mlda(c.doc_ptr, c.word_ids, V, K, alpha, beta, SEED, chunks=3)
    model.init_random()
    z = oracle.init_topics(c.T, K, SEED)
    for it in (1, 2):
        z = check_step(model, c, z, V, K, alpha, beta, SEED, it)
    model.close()


def test_streamed_edge_cases(mlda):
    """More chunks than documents, empty documents, long documents over few topics, and a saved
    state carried from a resident context into a streamed one."""
    base = corpus_synth.tiny(D=5, V=30, K=9, mean_len=12, seed=3)
    lens = np.diff(base.doc_ptr)
    new_lens = np.zeros(2 * len(lens) + 1, dtype=np.int64)
    new_lens[1::2] = lens                                   # empty documents in between

    class C:  # minimal corpus record
        pass
    c = C(); c.doc_ptr = np.concatenate([[0], np.cumsum(new_lens)]).astype(np.int64)
    c.word_ids = base.word_ids; c.T = base.T
    V, K, alpha, beta = 30, 9, 0.4, 0.02
    model = mlda.Mlda(c.doc_ptr, c.word_ids, V, K, alpha, beta, 11, chunks=16)
    model.init_random()
    z = oracle.init_topics(c.T, K, 11)
    for it in (1, 2):
        z = check_step(model, c, z, V, K, alpha, beta, 11, it)
    model.close()

    big = corpus_synth.tiny(D=4, V=40, K=50, mean_len=16500, seed=8)      # counts spread over many entries
    model = mlda.Mlda(big.doc_ptr, big.word_ids, 40, 50, 1.0, 0.01, SEED, chunks=3)
    model.init_random()
    z = oracle.init_topics(big.T, 50, SEED)
    z = check_step(model, big, z, 40, 50, 1.0, 0.01, SEED, 1)
    model.close()

    c1 = corpus_synth.generate("C1")
    cfg = c1.config
    args = (c1.doc_ptr, c1.word_ids, cfg.V, cfg.K, cfg.alpha, cfg.beta, SEED)
    a = mlda.Mlda(*args); a.init_random(); a.step(4)
    r = mlda.Mlda(*args); r.init_random(); r.step(2)
    s = mlda.Mlda(*args, chunks=4); s.set_assignments(r.assignments(), it=r.iteration); s.step(2)
    assert np.array_equal(s.assignments(), a.assignments())
    assert np.array_equal(s.word_topic(), a.word_topic())
    assert abs(s.loglik() - a.loglik()) <= 1e-9 * abs(a.loglik())
    for m in (a, r, s):
        m.close()

    empty = mlda.Mlda(np.zeros(3, dtype=np.int64), np.zeros(0, dtype=np.int32), 4, 3, 0.5, 0.01, 1, chunks=2)
    empty.init_random(); empty.step(2, loglik=True)
    assert empty.iteration == 2 and empty.doc_topic_nnz() == 0 and abs(empty.loglik()) < 1e-9
    empty.close()


def test_phi_cell_widths(mlda):
    """phi keeps 16-bit cells for words with fewer than 2^16 tokens and int32 rows for the
    others: words with 65535, 65536 and 70001 tokens, every token of a word on one topic (the
    largest value a 16-bit cell can take, and the first that needs the wide row), an odd K so
    that rows start in the middle of a dword; resident and streamed (cells added to by
    several chunks)."""
    V, K, alpha, beta = 5, 7, 0.5, 0.01
    word_counts = np.array([65535, 65536, 70001, 10, 0])
    rng = np.random.default_rng(5)
    word_ids = rng.permutation(np.repeat(np.arange(V, dtype=np.int32), word_counts))
    T = len(word_ids)
    lens = rng.multinomial(T, np.ones(400) / 400).astype(np.int64)

    class C:
        pass
    c = C(); c.word_ids = word_ids; c.T = T
    c.doc_ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    z_one = (c.word_ids % K).astype(np.uint16)              # word v entirely on topic v
    for chunks in (1, 3):
        say("phi cell widths, chunks", chunks)
        model = mlda.Mlda(c.doc_ptr, c.word_ids, V, K, alpha, beta, SEED, chunks=chunks)
        model.set_assignments(z_one, it=0)
        n_wk, _ = check_counts(model, c, z_one, V, K)
        assert n_wk[0, 0] == 65535 and n_wk[1, 1] == 65536 and n_wk[2, 2] == 70001
        n_wk, n_k = oracle.count_word_topic(c.word_ids, z_one, V, K)
        ll = oracle.loglik(c.doc_ptr, z_one, V, K, alpha, beta, n_wk, n_k)
        assert abs(model.loglik() - ll) <= LL_RTOL * abs(ll)
        z = z_one
        for it in (1, 2):
            z = check_step(model, c, z, V, K, alpha, beta, SEED, it)
        model.close()


@pytest.mark.parametrize("K", [1, 7, 8, 4095, 4096, 4097, 33001])
def test_phi_segment_edges(mlda, K):
    """phi and n_k of words whose tokens begin and end anywhere between the aligned eights that are read
    at a time, with rows that start in either half of a dword, whole words and words of several
    segments; totals counted beside phi (K <= 4096), in a launch of their own and in ranges of
    topics.  Three states in a row: the totals of one are cleared while the next is counted."""
    word_counts = np.array([1, 7, 0, 8, 9, 15, 16, 17, 1023, 16383, 1, 16384, 16385, 0, 33000, 3])
    V, alpha, beta = len(word_counts), 0.5, 0.01
    rng = np.random.default_rng(K)

    class C:
        pass
    c = C(); c.word_ids = rng.permutation(np.repeat(np.arange(V, dtype=np.int32), word_counts)); c.T = len(c.word_ids)
    lens = rng.multinomial(c.T, np.ones(300) / 300).astype(np.int64)
    c.doc_ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    for chunks in (1, 2):
        model = mlda.Mlda(c.doc_ptr, c.word_ids, V, K, alpha, beta, SEED, chunks=chunks)
        for _ in range(3):
            z = rng.integers(K, size=c.T).astype(np.uint16)
            model.set_assignments(z)
            check_counts(model, c, z, V, K)
        if K < 5000:
            check_step(model, c, z, V, K, alpha, beta, SEED, 1)
        model.close()


@pytest.mark.parametrize("K", [4097, 17000, 65535])
def test_phi_cells_of_changed_topics(mlda, K):
    """Rows of words of few tokens over many topics after a step and after assignments are installed: words of 1, 255, 256, 257
    and K / 64 tokens, one more, and one of two segments whose last has few; topics that stay, leave and come back."""
    most = K // 64
    word_counts = np.array([1, 0, 2, 64, min(most, 255), min(most, 256), min(most, 257), most, most + 1, 2 * 16384 + 3, 5])
    V, alpha, beta = len(word_counts), 50.0 / K, 0.01
    rng = np.random.default_rng(K)

    class C:
        pass
    c = C(); c.word_ids = rng.permutation(np.repeat(np.arange(V, dtype=np.int32), word_counts)); c.T = len(c.word_ids)
    c.doc_ptr = np.concatenate([[0], np.cumsum(rng.multinomial(c.T, np.ones(200) / 200))]).astype(np.int64)
    model = mlda.Mlda(c.doc_ptr, c.word_ids, V, K, alpha, beta, SEED)
    for it, few in enumerate((3, K)):
        z = rng.integers(few, size=c.T).astype(np.uint16)
        model.set_assignments(z, it=2 * it)
        for step in (1, 2):
            z = check_step(model, c, z, V, K, alpha, beta, SEED, 2 * it + step)
    model.close()


@pytest.mark.parametrize("K,longest", [(1500, 300), (453, 700), (1025, 132), (3072, 3071), (300, 500)])
def test_one_launch_rebuild_with_one_document_per_wave(mlda, K, longest):
    """phi and theta in one launch, four waves to a workgroup and a document to a wave, whose parts of LDS end in the middle of
    16 bytes: documents of 0 tokens to the longest, whose tokens beyond those in registers are an odd number of times four."""
    V, alpha, beta = 500, 50.0 / K, 0.01
    rng = np.random.default_rng(longest)
    lengths = rng.permutation(np.concatenate([np.full(20, longest), rng.integers(0, longest + 1, 60), np.full(60, longest // 4),
                                              [0, 1, 2, 127, 128, 129]]))

    class C:
        pass
    c = C(); c.T = int(lengths.sum())
    c.doc_ptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    c.word_ids = rng.integers(V, size=c.T).astype(np.int32)
    say("one document per wave", K, longest, "T", c.T)
    model = mlda.Mlda(c.doc_ptr, c.word_ids, V, K, alpha, beta, SEED)
    model.init_random()
    z = oracle.init_topics(c.T, K, SEED)
    for it in (1, 2):
        z = check_step(model, c, z, V, K, alpha, beta, SEED, it)
    model.close()


@pytest.mark.parametrize("K", [40, 3000])
def test_assignments_change_order_tile_by_tile(mlda, K, monkeypatch):
    """Both directions, tiles of every size up to the largest and one more, and a number of them that eight does not divide."""
    monkeypatch.setenv("MLDA_REORDER_BY_TILES", "0")
    V = 61
    rng = np.random.default_rng(K)
    per_word = np.concatenate([np.arange(1, V - 7), [255, 256, 257, 1023, 1024, 1025, 4097, 0]])
    words = rng.permutation(np.repeat(np.arange(V, dtype=np.int32), per_word))
    doc_ptr = np.concatenate([[0], np.sort(rng.choice(np.arange(1, len(words)), 90, replace=False)), [len(words)]]).astype(np.int64)
    for shape in ("1024,0", "64,64"):
        monkeypatch.setenv("MLDA_TILE_SHAPE", shape)
        model = mlda.Mlda(doc_ptr, words, V, K, 50.0 / K, 0.01, SEED)
        z = rng.integers(K, size=len(words)).astype(np.uint16)
        model.set_assignments(z)
        assert np.array_equal(model.assignments(), z)
        n_wk, n_k = oracle.count_word_topic(words, z, V, K)
        assert np.array_equal(model.word_topic(), n_wk) and np.array_equal(model.topic_totals(), n_k)
        model.close()


@pytest.mark.parametrize("run", ["16", "3", "1"])
@pytest.mark.parametrize("case", [c for c in EDGE_CASES if 2048 < c[3] <= 20000], ids=lambda c: c[0])
def test_large_k_in_runs(mlda, case, run, monkeypatch):
    """Small tiles one after the other in a workgroup, of which corpora of few words have none by themselves."""
    monkeypatch.setenv("MLDA_RUN_TILES", run)
    test_edge_shapes(mlda, case)


@pytest.mark.parametrize("chunks", [1, 2])
@pytest.mark.parametrize("K,mean_len", [(11439, 40), (11440, 40), (11440, 120), (26159, 40), (26159, 120), (26160, 120)])
def test_queued_tiles_at_the_edges_of_the_workgroups(mlda, K, mean_len, chunks, monkeypatch):
    """The last K of twelve waves and the first of sixteen, the last whose p* fits LDS and the first that is split; a word
    of more than 1,024 tokens, then small ones, sixteen tiles to a workgroup, so that p* is made from the word before's."""
    monkeypatch.setenv("MLDA_RUN_TILES", "16")
    V, alpha, beta = 400, 50.0 / K, 0.01
    c = corpus_synth.tiny(D=9600 // mean_len, V=V, K=K, mean_len=mean_len, seed=K)
    c.word_ids[: len(c.word_ids) // 6] = 7
    model = mlda.Mlda(c.doc_ptr, c.word_ids, V, K, alpha, beta, SEED, chunks=chunks)
    model.init_random()
    z = oracle.init_topics(c.T, K, SEED)
    for it in (1, 2):
        z = check_step(model, c, z, V, K, alpha, beta, SEED, it)
    model.close()


# (topics, lengths of the first documents, further documents of 3 tokens each)
RANKED_CASES = [("two_per_wave", 1000, [0, 1, 31, 32, 33, 127, 128, 129, 383, 384, 385, 1500, 4000, 0, 700], 60),
                ("two_per_wave_33", 33, [0, 1, 127, 128, 129, 383, 384, 385, 3000], 60),
                ("two_per_wave_1024", 1024, [2500, 1, 600, 3], 40),
                ("one_per_wave", 3000, [0, 1, 63, 64, 65, 127, 128, 129, 2175, 2176, 2177, 5000, 1153, 1152], 0),
                ("one_per_wave_2048", 2048, [4096, 128, 129, 2000, 0], 0),
                ("one_per_wave_largest", 65535, [3000, 1, 128, 1500, 300], 0)]


@pytest.mark.parametrize("case", RANKED_CASES, ids=[c[0] for c in RANKED_CASES])
def test_rows_by_ranks(mlda, case):
    """Rows of theta from topics' ranks: documents at the edges of what registers, the staged topics and
    one round of cells hold, rows of several rounds, counts of several entries in any of them,
    empty documents, an odd number of documents."""
    _, K, lens, short = case
    rng = np.random.default_rng(K)
    lens = np.array(lens + [3] * short, dtype=np.int64)

    class C:
        pass
    c = C(); V = 40
    c.doc_ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    c.T = int(lens.sum())
    c.word_ids = rng.integers(V, size=c.T).astype(np.int32)
    spread = rng.integers(K, size=c.T).astype(np.uint16)
    few = np.where(rng.random(c.T) < 0.7, rng.choice([0, K // 2, K - 1], size=c.T), spread).astype(np.uint16)
    for chunks in (1, 2):
        model = mlda.Mlda(c.doc_ptr, c.word_ids, V, K, 50.0 / K, 0.01, SEED, chunks=chunks)
        for it, z in enumerate((spread, few)):
            model.set_assignments(z, it=it)
            check_counts(model, c, z, V, K)
            check_step(model, c, z, V, K, 50.0 / K, 0.01, SEED, it + 1)
        model.close()


# (topics, lengths of the long documents, how many others and their tokens, empty documents): documents of more than 3,072
# tokens are rebuilt in a launch of their own (of one or sixteen waves each), which leaves fewer or more partial sums
# than the launch of the others that adds to them
UNEVEN_CASES = [("two_per_wave", 500, [3073, 3072, 3071, 9000, 30000], 300, 60, 3),
                ("one_per_wave", 5000, [3073, 3072, 2177, 2176, 5000, 30000], 100, 200, 5),
                ("one_per_wave_many_rounds", 40000, [30000, 60000, 3073], 300, 300, 0),
                ("counts_of_many_entries", 3, [3073, 60000], 200, 30, 1),
                ("few_others", 700, [3100] * 40, 3, 100, 80)]


@pytest.mark.parametrize("case", UNEVEN_CASES, ids=[c[0] for c in UNEVEN_CASES])
def test_rows_of_uneven_documents(mlda, case):
    name, K, long_docs, others, length, empty = case
    rng = np.random.default_rng(K)
    lens = rng.permutation(np.array(long_docs + [length] * others + [0] * empty, dtype=np.int64))

    class C:
        pass
    c = C(); V = 50
    c.doc_ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    c.T = int(lens.sum())
    c.word_ids = rng.integers(V, size=c.T).astype(np.int32)
    z = rng.integers(K, size=c.T).astype(np.uint16)
    for chunks in (1, 2):
        say(name, "chunks", chunks)
        model = mlda.Mlda(c.doc_ptr, c.word_ids, V, K, 50.0 / K, 0.01, SEED, chunks=chunks)
        model.set_assignments(z)
        check_counts(model, c, z, V, K)
        check_step(model, c, z, V, K, 50.0 / K, 0.01, SEED, 1)
        if chunks == 1 and K < 1024:        # the sums of row entries, in the bytes
            row_ptr, _, counts = oracle.doc_topic_csr(c.doc_ptr, z, K)
            entries = np.array([(-(-counts[a:b] // 15)).sum() for a, b in zip(row_ptr[:-1], row_ptr[1:])])
            tiles = np.ceil(np.bincount(c.word_ids, minlength=V) / 1024).sum()
            assert model.sampler_bytes()[-1] == 16.0 * c.T + 2.0 * float((lens * entries).sum()) + K * 2.0 * tiles
        model.close()


@pytest.mark.parametrize("K", [5000, 40000])
def test_one_long_document_costs_what_its_tokens_do(mlda, K):
    """The theta rebuild of 3e6 tokens in documents of 300 takes longer with one document of 60,000 among them, but by
    no more than one wave that reads each of its tokens once: 4.7 ns a token, and as much again to spare."""
    V, longest = 500, 60000

    def rebuild_ms(lens):
        doc_ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
        words = np.random.default_rng(1).integers(V, size=int(doc_ptr[-1])).astype(np.int32)
        model = mlda.Mlda(doc_ptr, words, V, K, 50.0 / K, 0.01, SEED)
        model.init_random(); model.step(3)
        ms = model.timing()[:, 2].min()
        model.close()
        return ms
    even = rebuild_ms(np.full(10000, 300))
    uneven = rebuild_ms(np.concatenate([np.full(5000, 300), [longest], np.full(4800, 300)]))
    say(K, "theta rebuild", even, "ms even,", uneven, "ms uneven")
    assert uneven <= even + 2 * 4.7e-6 * longest


@pytest.mark.parametrize("how", ["own_stream", "stream_per_thread", "streamed"])
def test_large_transfers(mlda, how):
    """Transfers of 8 MB and more go through eight pinned pieces of 2 MB, each with a thread of its own:
    18 MB of assignments and row values and 9 MB of word counts here, so that a thread has several
    pieces and the last one is short; a document of 70,000 tokens of one topic (counts of more than
    16 bits are fetched in two halves), a word with 32-bit counts, empty documents.  The handle
    hipStreamPerThread names another stream in every thread."""
    import torch
    V, K, alpha, beta = 70000, 64, 0.5, 0.01
    rng = np.random.default_rng(7)
    lens = rng.integers(0, 200, size=92000).astype(np.int64)
    lens[::1000] = 0
    lens[40000] = 70000

    class C:  # minimal corpus record
        pass
    c = C(); c.doc_ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    c.T = int(lens.sum())
    assert 9.0e6 < c.T < 9.4e6 and c.T % (1 << 20) != 0
    c.word_ids = rng.integers(V, size=c.T).astype(np.int32)
    c.word_ids[rng.integers(c.T, size=100000)] = 3
    z = rng.integers(K, size=c.T).astype(np.uint16)
    z[c.doc_ptr[40000]:c.doc_ptr[40001]] = 5
    stream = torch.cuda.ExternalStream(2) if how == "stream_per_thread" else torch.cuda.current_stream()
    with torch.cuda.stream(stream):
        model = mlda.Mlda(c.doc_ptr, c.word_ids, V, K, alpha, beta, SEED, chunks=2 if how == "streamed" else 1)
        assert how != "stream_per_thread" or model.stream.cuda_stream == 2
        model.set_assignments(z)
        assert np.array_equal(model.assignments(), z)
        check_counts(model, c, z, V, K)
        check_step(model, c, z, V, K, alpha, beta, SEED, 1)
        model.close()


def test_getters_leave_nothing_on_the_stream(mlda):
    """A getter synchronises the stream, whichever way its bytes take: of 16 MB and 9 MB, and of few."""
    V, K = 70000, 64
    rng = np.random.default_rng(5)
    T = (8 << 20) + 4321
    doc_ptr = np.append(np.arange(0, T, 100), T).astype(np.int64)
    model = mlda.Mlda(doc_ptr, rng.integers(V, size=T).astype(np.int32), V, K, 0.5, 0.01, SEED)
    model.init_random()
    busy = {"assignments": 0, "word_topic": 0, "doc_topic_csr": 0, "topic_totals": 0, "loglik": 0}
    for _ in range(20):
        for name in busy:
            getattr(model, name)()
            busy[name] += not model.stream.query()
    say(busy)
    model.close()
    assert not any(busy.values())


def test_empty_corpus(mlda):
    doc_ptr = np.zeros(4, dtype=np.int64)
    model = mlda.Mlda(doc_ptr, np.zeros(0, dtype=np.int32), 5, 3, 0.5, 0.01, 1)
    model.init_random()
    model.step(2)
    assert model.iteration == 2 and len(model.assignments()) == 0
    assert model.word_topic().sum() == 0 and model.doc_topic_nnz() == 0
    row_ptr, topics, counts = model.doc_topic_csr()
    assert np.array_equal(row_ptr, np.zeros(4)) and len(topics) == 0
    # all counts zero: every lgamma difference vanishes
    assert abs(model.loglik()) < 1e-9
    model.close()


def test_deterministic_and_resumable(mlda):
    """Two runs are bit-identical; 6 iterations == 3 + export + new context + import + 3."""
    c = corpus_synth.generate("C1")
    cfg = c.config
    args = (c.doc_ptr, c.word_ids, cfg.V, cfg.K, cfg.alpha, cfg.beta, SEED)
    a = mlda.Mlda(*args); a.init_random(); a.step(6)
    b = mlda.Mlda(*args); b.init_random(); b.step(6)
    za = a.assignments()
    assert np.array_equal(za, b.assignments())
    assert a.loglik() == b.loglik()
    r = mlda.Mlda(*args); r.init_random(); r.step(3)
    saved, it = r.assignments(), r.iteration
    r.close()
    r2 = mlda.Mlda(*args); r2.set_assignments(saved, it=it); r2.step(3)
    assert np.array_equal(r2.assignments(), za) and r2.iteration == 6
    assert np.array_equal(r2.word_topic(), a.word_topic())
    # another seed is another chain
    d = mlda.Mlda(*args[:-1], SEED + 1); d.init_random(); d.step(1)
    assert not np.array_equal(d.assignments()[:1000], za[:1000])
    for m in (a, b, r2, d):
        m.close()


def test_step_with_loglik_flag_and_timing(mlda):
    c = corpus_synth.generate("C1")
    cfg = c.config
    model = mlda.Mlda(c.doc_ptr, c.word_ids, cfg.V, cfg.K, cfg.alpha, cfg.beta, SEED)
    model.init_random()
    ll0 = model.loglik()
    model.step(4, loglik=True)
    ms = model.timing()
    assert ms.shape == (4, 4) and np.all(ms[:, :3] > 0) and np.all(ms < 1000)
    z = model.assignments()
    n_wk, n_k = oracle.count_word_topic(c.word_ids, z, cfg.V, cfg.K)
    ll = oracle.loglik(c.doc_ptr, z, cfg.V, cfg.K, cfg.alpha, cfg.beta, n_wk, n_k)
    assert abs(model.loglik() - ll) <= LL_RTOL * abs(ll)
    assert model.loglik() > ll0
    # the algorithmic byte count of each launch follows its definition: the state a launch
    # samples from is the one before it
    per_word = np.bincount(c.word_ids, minlength=cfg.V)
    n_tiles = int(np.ceil(per_word / 1024).sum())
    n_wide_tiles = int(np.ceil(per_word[per_word >= 2**16] / 1024).sum())   # int32 rows of phi
    lens = np.diff(c.doc_ptr)

    def row_entries(assignments):
        """Entries of every theta row as the byte count takes them: for K < 1024 of counts up to 15,
        so a larger count takes several, whatever the layout in use."""
        row_ptr, _, counts = oracle.doc_topic_csr(c.doc_ptr, assignments, cfg.K)
        per_topic = -(-counts.astype(np.int64) // 15)
        return np.array([per_topic[row_ptr[d]:row_ptr[d + 1]].sum() for d in range(len(lens))])

    assert cfg.K < 1024
    before = row_entries(model.assignments())
    model.step(2)
    mid = row_entries(oracle.iteration(c.doc_ptr, c.word_ids, z, cfg.V, cfg.K, cfg.alpha, cfg.beta, SEED, 5))
    got = model.sampler_bytes()
    assert (before > np.diff(oracle.doc_topic_csr(c.doc_ptr, z, cfg.K)[0])).any()     # some counts are spread
    for entries, b in zip((before, mid), got):
        want = (16.0 * c.T + 2.0 * float((lens * entries).sum())
                + cfg.K * (2.0 * n_tiles + 2.0 * n_wide_tiles))
        assert b == want
    assert len(got) == 2
    model.close()


# (name, K, document lengths as (how many, tokens)): every way a row of theta is built for K <= 2048.
# Counts are far beyond 15 (K < 1024) and 16,383 (K >= 1024).
BYTES_CASES = [
    ("four_byte_rows_two_documents_per_wave", 24,   [(60, 110)]),
    ("four_byte_rows_one_wave",               24,   [(40, 600)]),
    ("four_byte_rows_sixteen_waves",          50,   [(4, 6000)]),
    ("four_byte_rows_wide_counters",          5,    [(2, 70000)]),
    ("two_byte_rows_long_count",              1500, [(2000, 300), (1, 20000)]),
    ("two_byte_rows_wide_counters",           2048, [(2000, 1500), (1, 66000)]),
    ("six_bits_two_documents_per_wave",       60,   [(200, 150)]),
    ("six_bits_one_wave",                     300,  [(30, 1500)]),
]


@pytest.mark.parametrize("case", BYTES_CASES, ids=[c[0] for c in BYTES_CASES])
def test_sampler_bytes_in_every_row_layout(mlda, case):
    """The algorithmic bytes are those of entries of up to 15 tokens (2 bytes, K < 1024) or 16,383
    (4 bytes), whatever the entries of the layout in use hold."""
    name, K, docs = case
    V, alpha, beta = 60, 50.0 / K, 0.01
    lens = np.concatenate([np.full(n, length, dtype=np.int64) for n, length in docs])
    doc_ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    rng = np.random.default_rng(len(name))
    words = rng.integers(V, size=int(lens.sum())).astype(np.int32)
    z = rng.integers(K, size=len(words)).astype(np.uint16)
    z[doc_ptr[-2]:doc_ptr[-1]] = K // 2           # the last document sits in one topic
    model = mlda.Mlda(doc_ptr, words, V, K, alpha, beta, SEED)
    model.set_assignments(z)
    model.step(1)
    row_ptr, _, counts = oracle.doc_topic_csr(doc_ptr, z, K)
    entries = np.add.reduceat(-(-counts.astype(np.int64) // (15 if K < 1024 else 16383)), row_ptr[:-1])
    per_word = np.bincount(words, minlength=V)
    want = (16.0 * len(words) + (2.0 if K < 1024 else 4.0) * float((lens * entries).sum())
            + K * (2.0 * np.ceil(per_word / 1024).sum() + 2.0 * np.ceil(per_word[per_word >= 2**16] / 1024).sum()))
    assert model.sampler_bytes()[-1] == want
    model.close()


def test_sampler_bytes_with_runs_of_small_words(mlda):
    """K > 2048: the words of at most 1024 tokens are sampled in runs of 16 and count 6 bytes per
    token instead of a row of phi each, but for the first word of every run."""
    D, V, K = 300, 500, 4000
    c = corpus_synth.tiny(D=D, V=V, K=K, mean_len=200, seed=21, name="runs")
    alpha, beta = 50.0 / K, 0.01
    model = mlda.Mlda(c.doc_ptr, c.word_ids, V, K, alpha, beta, SEED)
    model.init_random()
    z = oracle.init_topics(c.T, K, SEED)
    z = check_step(model, c, z, V, K, alpha, beta, SEED, 1)
    row_ptr, _, _ = oracle.doc_topic_csr(c.doc_ptr, oracle.init_topics(c.T, K, SEED), K)
    lens = np.diff(c.doc_ptr)
    per_word = np.bincount(c.word_ids, minlength=V)
    per_word = per_word[per_word > 0]
    n_tiles = int(np.ceil(per_word / 4096).sum())
    in_runs = per_word[per_word <= 1024]
    assert 16 < len(in_runs) < len(per_word)          # runs, and words outside them
    staged_rows = n_tiles - len(in_runs) + -(-len(in_runs) // 16)
    want = (16.0 * c.T + 4.0 * float((lens * np.diff(row_ptr)).sum())
            + K * 2.0 * staged_rows + 6.0 * float(in_runs.sum()))
    assert model.sampler_bytes()[-1] == want
    model.close()


def test_device_side_argument_errors(mlda):
    import torch
    lib = mlda.load_library()
    c = corpus_synth.tiny(D=10, V=20, K=4, mean_len=5, seed=1)
    model = mlda.Mlda(c.doc_ptr, c.word_ids, 20, 4, 0.5, 0.01, 1)
    with pytest.raises(mlda.MldaError) as e:           # no state yet
        model.step(1)
    assert e.value.code == -1
    with pytest.raises(mlda.MldaError):
        model.assignments()
    with pytest.raises(mlda.MldaError):                # topic >= K
        model.set_assignments(np.full(c.T, 4, dtype=np.uint16))
    model.init_random()
    with pytest.raises(mlda.MldaError):
        model.step(-1)
    model.close()
    bad_words = c.word_ids.copy(); bad_words[3] = 20
    with pytest.raises(mlda.MldaError) as e:
        mlda.Mlda(c.doc_ptr, bad_words, 20, 4, 0.5, 0.01, 1)
    assert e.value.code == -1 and "word id" in str(e.value)
    # host memory handed in as the device workspace
    ctx = ctypes.c_void_p()
    host = np.zeros(1 << 22, dtype=np.uint8)
    addr = (host.ctypes.data + 255) // 256 * 256
    rc = lib.mlda_create(ctypes.addressof(ctx), c.doc_ptr.ctypes.data, c.word_ids.ctypes.data,
                         10, 20, 4, 0.5, 0.01, 1, ctypes.c_void_p(addr), (1 << 22) - 256, None)
    assert rc == -1 and b"not device memory" in lib.mlda_last_error()
    # every K up to 65,535 is served
    big_k = 60000
    model = mlda.Mlda(c.doc_ptr, c.word_ids, 20, big_k, 0.5, 0.01, 1)
    model.close()
