"""Edges of the kernels' tiles and of the rules that choose between them, each against the oracle."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_common import log, oracle_side, row_rel_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def w2v():
    import paper_1606_07822_amd as m
    return m


def to_dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# ------------------------------------------------------------- Huffman
# The merge gives each of up to 128 workgroups chunks of 2,048 picks of a generation: one workgroup, a chunk for
# every workgroup, and more chunks than workgroups (a generation of equal counts is as long as the vocabulary);
# codes that fill the points' staging space (32 turns on average) and exceed it.
@pytest.mark.parametrize("V,kind", [(128 * 2048, "equal"), (128 * 2048 + 1, "equal"), (300_001, "few"),
                                    (524_289, "few"), (700_000, "wide"), (60, "deep"), (256 * 3 + 62, "deep")])
def test_huffman_across_workgroups_bit_exact(w2v, V, kind):
    rng = np.random.default_rng(V)
    if kind == "equal":
        counts = np.full(V, 7)
    elif kind == "few":
        counts = rng.choice([5, 6, 11, 5000], V, p=[0.6, 0.3, 0.0999, 0.0001])
    elif kind == "wide":
        counts = np.floor(2.0 ** rng.uniform(0, 36, V)) + 1
    else:   # 60 levels from Fibonacci counts, the rest of the words at the bottom of the tree
        fib = [1 << 10, 1 << 10]
        while len(fib) < 44:
            fib.append(fib[-1] + fib[-2])
        counts = np.concatenate([np.array(fib[2:], np.int64) * max(1, V // 1024 + 1), np.ones(V - 42)])
    counts = np.sort(counts.astype(np.int64))[::-1].copy()
    t, o = w2v.build_huffman(to_dev(counts)), oracle.build_huffman(counts)
    np.testing.assert_array_equal(t.codelen.cpu().numpy(), o.codelen)
    np.testing.assert_array_equal(t.code.cpu().numpy().view(np.uint64), o.code)
    np.testing.assert_array_equal(t.point_off.cpu().numpy(), o.point_off)
    np.testing.assert_array_equal(t.points.cpu().numpy(), o.points)
    assert t.max_len == int(o.codelen.max())


@pytest.mark.parametrize("V", [66, 74, 88])
def test_huffman_too_deep_at_any_generation_is_an_error(w2v, V):
    fib = [1, 1]
    while len(fib) < V:
        fib.append(fib[-1] + fib[-2])
    with pytest.raises(w2v.W2VError) as e:
        w2v.build_huffman(to_dev(np.array(fib[::-1], np.int64)))
    assert e.value.code == w2v.W2V_E_RANGE


# Counts (runs of multiples of 2^60) whose sums pass 2^63: the merge's queues are no longer ascending, some inner
# nodes are never taken, and the paths of the words below them (a model of the merge on the CPU: 4 to 9 of them,
# whichever of two writers of another entry wins) end there. They are refused, and nothing is read through them.
@pytest.mark.parametrize("runs", [
    [(7, 6), (6, 7), (5, 4), (4, 3), (3, 4), (2, 2), (1, 5)], [(7, 3), (6, 1), (5, 4), (4, 7), (3, 8), (2, 4), (1, 5)],
    [(7, 4), (6, 7), (5, 6), (4, 3), (3, 4), (2, 6), (1, 3)],
])
def test_huffman_counts_past_63_bits_are_an_error(w2v, runs):
    counts = np.concatenate([np.full(n, x << 60, np.int64) for x, n in runs])
    with pytest.raises(w2v.W2VError) as e:
        w2v.build_huffman(to_dev(counts))
    assert e.value.code == w2v.W2V_E_RANGE


# ------------------------------------------------------------- narrow rows
# Skip-gram rows of up to 128 floats on the store-only walk: the widest and narrowest row of each variant, every
# write policy that takes it, no subsampling over 1,000 words (repeated words in most windows), short documents, a
# large cache, windows above 5. The bar is the one of the other single-worker tests: sums in another order and the
# fast sigmoid, carried through the updates.
@pytest.mark.parametrize("name,sample,dim,win,wp,k,doc_len", [
    ("tiny_sg_v1k_d50", 0.0, 50, 2, 5, 31, 1000), ("tiny_sg_v1k_d50", 0.0, 64, 5, 7, 31, 1000),
    ("tiny_sg_v1k_d50", 0.0, 65, 5, 5, 31, 1000), ("tiny_sg_v1k_d50", 0.0, 1, 3, 15, 7, 1000),
    ("tiny_sg_v1k_d50", 0.0, 128, 2, 7, 0, 1000), ("tiny_sg_v1k_d50", 0.0, 100, 4, 1, 0, 7),
    ("tiny_sg_v1k_d50", 0.0, 33, 1, 5, 31, 3), ("tiny_sg_v1k_d50", 0.0, 100, 5, 5, 31, 129),
    ("sg_v30k_d100", 1e-3, 100, 5, 5, 31, 1000), ("sg_v30k_d100", 1e-3, 127, 3, 7, 31, 1000),
    ("sg_v30k_d100", 1e-3, 100, 5, 5, 120, 1000), ("sg_v30k_d100", 1e-3, 100, 6, 5, 31, 1000),
    ("sg_v30k_d100", 1e-3, 64, 10, 7, 31, 1000),
])
def test_narrow_rows_single_worker_matches_oracle(w2v, name, sample, dim, win, wp, k, doc_len):
    log(f"narrow rows {name} dim={dim} window={win} write_policy={wp} k={k} doc_len={doc_len}")
    s = oracle_side(name)
    voc = w2v.build_vocab(to_dev(s.tok), s.w.vocab, s.w.min_count)
    tree = w2v.build_huffman(voc.vocab_counts)
    tv = s.tv[:3001]
    syn0, syn1 = synth.init_weights(s.voc.V, dim, syn1_scale=0.5 / dim)
    a0, a1 = syn0.copy(), syn1.copy()
    op = oracle.params(s.voc.V, dim, window=win, sample=sample, train_words=s.voc.train_words,
                       corpus_tokens=s.tv.size, cache_k=k, flush_every=10, order=1, doc_len=doc_len)
    ost = oracle.train(a0, a1, s.tree, tv, op)
    model = w2v.make_model(syn0, syn1, voc, tree, stride=(dim + 3) // 4 * 4, pad_value=float("nan"))
    p = w2v.Params(window=win, sample=sample, corpus_tokens=s.tv.size, cache_k=k, flush_every=10, workers=1,
                   write_policy=wp, doc_len=doc_len)
    st = w2v.train_hs_epoch(model, to_dev(tv), p).cpu().numpy()
    assert list(st) == list(ost)
    g0, g1 = (t.cpu().numpy() for t in model.vectors())
    assert row_rel_err(g0, a0) <= 1e-4
    assert row_rel_err(g1[:s.voc.V - 1], a1) <= 1e-4


# Text without subsampling at full occupancy: thousands of wavefronts train the most frequent words at once, and what
# each adds to their rows was computed without the others' latest. The longer a wavefront holds a change back, the
# lower the learning rate at which the sums overshoot: with a change kept until its position leaves the window these
# rates diverge (at window 5 from 0.016 on), with a write per centre they are two thirds of the limit (0.038 and
# 0.048), and stored rows (write_policy 7) have none. The untrained model's log-likelihood is beaten by 0.3 or more.
@pytest.mark.parametrize("V,dim,win,wp,alpha", [(50, 50, 5, 5, 0.025), (300, 100, 3, 5, 0.03), (1000, 100, 5, 7, 0.05),
                                                (50, 50, 5, 7, 0.05)])
def test_unsubsampled_text_trains_at_full_occupancy(w2v, V, dim, win, wp, alpha):
    log(f"unsubsampled V={V} dim={dim} window={win} write_policy={wp} alpha={alpha}")
    n, g = 4_000_000, torch.Generator(device="cuda").manual_seed(3)
    prob = 1.0 / torch.arange(1, V + 1, device="cuda", dtype=torch.float64)
    prob /= prob.sum()
    tok = torch.searchsorted(torch.cumsum(prob, 0), torch.rand(n, generator=g, device="cuda", dtype=torch.float64))
    # a document's topic, one word of each 20 neighbouring ranks, takes half of its tokens
    topic = torch.randint(20, (n // 1000,), generator=g, device="cuda").repeat_interleave(1000)
    tok = torch.where(torch.rand(n, generator=g, device="cuda") < 0.5, tok // 20 * 20 + topic, tok).clamp_(max=V - 1).int()
    voc = w2v.Vocab(None, None, (prob * n).long() + 5, None, V, int(((prob * n).long() + 5).sum()), None)
    syn0, syn1 = synth.init_weights(V, dim)
    model = w2v.make_model(syn0, syn1, voc, w2v.build_huffman(voc.vocab_counts))

    def ll():
        s, pairs, _ = w2v.hs_loglik(model, tok[:200_000], w2v.Params(window=win, seed=4))
        return s / pairs

    before = ll()
    w2v.train_hs_epoch(model, tok, w2v.Params(window=win, alpha0=alpha, write_policy=wp))
    after = ll()
    log(f"  untrained {before:.4f} trained {after:.4f} largest {float(model.syn0.abs().max()):.2f}")
    assert all(bool(torch.isfinite(t).all()) for t in model.vectors())
    assert after > before + 0.2


# Word rows kept across centres at 129 to 256 floats: the sixteen-wavefront variant, and the twelve-wavefront one
# where the cache (or the cache and the stash) leaves no room for it.
@pytest.mark.parametrize("arch", [0, 1])
@pytest.mark.parametrize("dim,k,stash", [(129, 31, 0), (256, 61, 0), (200, 64, 0), (256, 31, 1), (200, 56, 1)])
def test_word_span_variants_single_worker_match_oracle(w2v, arch, dim, k, stash):
    log(f"span arch={arch} dim={dim} k={k} stash={stash}")
    s = oracle_side("tiny_sg_v1k_d50")
    voc = w2v.build_vocab(to_dev(s.tok), s.w.vocab, s.w.min_count)
    tree = w2v.build_huffman(voc.vocab_counts)
    tv = s.tv[:2003]
    syn0, syn1 = synth.init_weights(s.voc.V, dim, syn1_scale=0.5 / dim)
    a0, a1 = syn0.copy(), syn1.copy()
    op = oracle.params(s.voc.V, dim, window=5, sample=0.0, train_words=s.voc.train_words, arch=arch,
                       corpus_tokens=s.tv.size, cache_k=k, flush_every=10, order=1)
    ost = oracle.train(a0, a1, s.tree, tv, op)
    model = w2v.make_model(syn0, syn1, voc, tree)
    p = w2v.Params(window=5, sample=0.0, corpus_tokens=s.tv.size, cache_k=k, flush_every=10, workers=1, arch=arch,
                   write_policy=15, span_stash=stash, stash_from=0)
    assert w2v.train_word_span(model, p) == 5
    st = w2v.train_hs_epoch(model, to_dev(tv), p).cpu().numpy()
    assert list(st) == list(ost)
    g0, g1 = (t.cpu().numpy() for t in model.vectors())
    assert row_rel_err(g0, a0) <= 1e-4
    assert row_rel_err(g1[:s.voc.V - 1], a1) <= 1e-4


# The sixteen-wavefront variants (129 to 256 floats) run where the wavefronts fill the chip and the training is long
# (2e8 raw tokens by its parameters); up to 128 floats the same launch runs the variants that short texts take. One document of at most 128 tokens is one work unit, so one of
# 4,096 wavefronts trains it and the result is the sequential one (write-backs that add the change: the other
# workgroups have none).
@pytest.mark.parametrize("arch,dim,win,wp,k,stash", [
    (0, 65, 5, 5, 31, 0), (0, 100, 2, 7, 31, 0), (0, 128, 4, 7, 0, 0), (0, 129, 5, 15, 31, 0), (0, 256, 5, 15, 31, 1),
    (0, 200, 3, 15, 64, 0), (1, 129, 5, 15, 31, 0), (1, 256, 2, 15, 31, 1), (1, 200, 5, 15, 31, 0),
])
def test_sixteen_wavefronts_single_unit_matches_oracle(w2v, arch, dim, win, wp, k, stash):
    log(f"sixteen wavefronts arch={arch} dim={dim} window={win} write_policy={wp} k={k} stash={stash}")
    s = oracle_side("tiny_sg_v1k_d50")
    voc = w2v.build_vocab(to_dev(s.tok), s.w.vocab, s.w.min_count)
    tree = w2v.build_huffman(voc.vocab_counts)
    tv = s.tv[:128]
    syn0, syn1 = synth.init_weights(s.voc.V, dim, syn1_scale=0.5 / dim)
    a0, a1 = syn0.copy(), syn1.copy()
    op = oracle.params(s.voc.V, dim, window=win, sample=0.0, train_words=s.voc.train_words, arch=arch,
                       corpus_tokens=200_000_000, cache_k=k, flush_every=10, order=1, doc_len=128)
    ost = oracle.train(a0, a1, s.tree, tv, op)
    model = w2v.make_model(syn0, syn1, voc, tree)
    p = w2v.Params(window=win, sample=0.0, corpus_tokens=200_000_000, cache_k=k, flush_every=10, flush_policy=0,
                   workers=4096, arch=arch, write_policy=wp, doc_len=128, span_stash=stash, stash_from=0)
    st = w2v.train_hs_epoch(model, to_dev(tv), p).cpu().numpy()
    assert list(st) == list(ost)
    if dim > 128:   # 64 cached rows leave no room for sixteen wavefronts' records
        assert w2v.last_train_launch() == (-(-4096 // (12 if k == 64 else 16)), 4096)
    g0, g1 = (t.cpu().numpy() for t in model.vectors())
    assert row_rel_err(g0, a0) <= 1e-4
    assert row_rel_err(g1[:s.voc.V - 1], a1) <= 1e-4


# A short training keeps twelve wavefronts a workgroup: with sixteen, 4,096 at once, the stored word rows overwrite so
# much of each other's changes that the model of this text gains 0.72 (skip-gram) and 0.21 (CBOW) of what 3,072 give.
@pytest.mark.parametrize("arch", [0, 1])
def test_short_training_learns_as_with_twelve_wavefronts(w2v, arch):
    log(f"short training arch={arch}")
    V, dim, n, g = 100_000, 200, 8_000_000, torch.Generator(device="cuda").manual_seed(3)
    prob = 1.0 / torch.arange(1, V + 1, device="cuda", dtype=torch.float64)
    prob /= prob.sum()
    tok = torch.searchsorted(torch.cumsum(prob, 0), torch.rand(n, generator=g, device="cuda", dtype=torch.float64))
    topic = torch.randint(20, (n // 1000,), generator=g, device="cuda").repeat_interleave(1000)
    tok = torch.where(torch.rand(n, generator=g, device="cuda") < 0.5, tok // 20 * 20 + topic, tok).clamp_(max=V - 1).int()
    counts = (prob * n).long() + 5
    voc = w2v.Vocab(None, None, counts, None, V, int(counts.sum()), None)
    syn0, syn1 = synth.init_weights(V, dim)
    tree = w2v.build_huffman(counts)
    settings = dict(window=5, sample=1e-5, arch=arch)

    def gain(workers):
        model = w2v.make_model(syn0, syn1, voc, tree)
        p = w2v.Params(alpha0=0.05 if arch == 1 else 0.025, write_policy=15, workers=workers, **settings)
        ll = []
        for train in (False, True):
            if train:
                w2v.train_hs_epoch(model, tok, p)
            s, terms, _ = w2v.hs_loglik(model, tok[:300_000], w2v.Params(seed=4, **settings))
            ll.append(s / terms)
        log(f"  workers {workers}: {ll[0]:.4f} -> {ll[1]:.4f}, {w2v.last_train_launch()}")
        return ll[1] - ll[0]

    assert gain(0) >= 0.9 * gain(3072)


# ------------------------------------------------------------- synchronous mode
# Every variant (rows of up to 64, 128, 256, 320, 512 and 1024 floats) at both ends of its range, windows that
# take one group of words and several (12, 8 or 4 words a group), single-word windows, batches of one and of
# more than one centre, and a last batch that is not full. The sums are exact on both sides; the bar is the
# other synchronous tests'.
@pytest.mark.parametrize("dim,win,batch", [(1, 1, 1), (64, 6, 100), (65, 10, 256), (128, 7, 33), (129, 4, 256),
                                           (256, 10, 64), (257, 5, 256), (320, 2, 100), (321, 3, 64), (512, 10, 128),
                                           (513, 2, 64), (1024, 9, 50)])
def test_sync_variants_match_oracle(w2v, dim, win, batch):
    log(f"sync dim={dim} window={win} batch={batch}")
    s = oracle_side("tiny_sg_v1k_d50")
    voc = w2v.build_vocab(to_dev(s.tok), s.w.vocab, s.w.min_count)
    tree = w2v.build_huffman(voc.vocab_counts)
    tv = s.tv[:1501]
    syn0, syn1 = synth.init_weights(s.voc.V, dim, syn1_scale=0.5 / dim)
    a0, a1 = syn0.copy(), syn1.copy()
    op = oracle.params(s.voc.V, dim, window=win, sample=1e-3, train_words=s.voc.train_words,
                       corpus_tokens=s.tv.size, sync_batch=batch)
    ost = oracle.train_sync(a0, a1, s.tree, tv, op, n_batches=-1)
    model = w2v.make_model(syn0, syn1, voc, tree, stride=(dim + 3) // 4 * 4, pad_value=float("nan"))
    p = w2v.Params(window=win, sample=1e-3, corpus_tokens=s.tv.size, mode=1, sync_batch=batch,
                   cache_k=0)
    st = w2v.train_hs_epoch(model, to_dev(tv), p).cpu().numpy()
    assert list(st) == list(ost)
    g0, g1 = (t.cpu().numpy() for t in model.vectors())
    assert row_rel_err(g0, a0) <= 1e-4
    assert row_rel_err(g1[:s.voc.V - 1], a1) <= 1e-4


# A batch of more centres than one launch's threads can number (2^32, 512 a centre): the sums of all of them are
# taken against the model at the batch's start.
def test_sync_batch_larger_than_a_launch_matches_oracle(w2v):
    V, dim, n = 60, 4, (1 << 23) + 5
    counts = np.sort(np.random.default_rng(1).integers(100, 10_000, V))[::-1].astype(np.int64)
    tv = np.random.default_rng(2).integers(0, V, n).astype(np.int32)
    voc = w2v.Vocab(None, None, to_dev(counts), None, V, int(counts.sum()), None)
    syn0, syn1 = synth.init_weights(V, dim, syn1_scale=0.1)
    a0, a1 = syn0.copy(), syn1.copy()
    op = oracle.params(V, dim, window=1, sample=0.0, train_words=int(counts.sum()), corpus_tokens=n, sync_batch=1 << 30)
    ost = oracle.train_sync(a0, a1, oracle.build_huffman(counts), tv, op, n_batches=-1)
    model = w2v.make_model(syn0, syn1, voc, w2v.build_huffman(voc.vocab_counts))
    p = w2v.Params(window=1, sample=0.0, corpus_tokens=n, mode=1, sync_batch=1 << 30, cache_k=0)
    st = w2v.train_hs_epoch(model, to_dev(tv), p).cpu().numpy()
    assert list(st) == list(ost) and st[2] == n
    g0, g1 = (t.cpu().numpy() for t in model.vectors())
    assert row_rel_err(g0, a0) <= 1e-4
    assert row_rel_err(g1[:V - 1], a1) <= 1e-4


# ------------------------------------------------------------- log-likelihood
# Rows that end inside, at and just past a 64-column tile and a panel of 512 columns, rows that are not a
# multiple of four floats (with NaN behind them), windows that take one and several groups of words, documents
# shorter and longer than a unit of eight centres, and paths past 32 nodes (a step's limit). The bar is the one
# of the other log-likelihood tests: 32-bit dot products (skip-gram), 64-bit everything (CBOW).
@pytest.mark.parametrize("arch", [0, 1])
@pytest.mark.parametrize("dim,win,doc_len,deep", [(1, 1, 1000, False), (63, 5, 9, False), (64, 4, 1000, False),
                                                  (66, 10, 1000, True), (128, 5, 7, False), (131, 6, 1000, False),
                                                  (256, 5, 1000, True), (301, 9, 1000, False), (320, 5, 129, False),
                                                  (323, 3, 1000, True), (512, 10, 1000, False),
                                                  (513, 5, 1000, False), (1023, 2, 1000, True), (1024, 4, 100, False)])
def test_loglik_variants_match_oracle(w2v, arch, dim, win, doc_len, deep):
    log(f"loglik arch={arch} dim={dim} window={win} doc_len={doc_len} deep={deep}")
    rng = np.random.default_rng(dim)
    if deep:   # 45 levels: Fibonacci counts over the last of them
        fib = [1, 1]
        while len(fib) < 45:
            fib.append(fib[-1] + fib[-2])
        counts = np.array(fib[::-1], np.int64)
    else:
        counts = np.sort(rng.integers(5, 5000, 700))[::-1].astype(np.int64)
    V = counts.size
    tv = rng.integers(-1, V, 1203).astype(np.int32)
    otree, tree = oracle.build_huffman(counts), w2v.build_huffman(to_dev(counts))
    syn0, syn1 = synth.init_weights(V, dim, syn1_scale=3.0 / dim ** 0.5)
    syn0 = syn0 * np.float32(dim)
    voc = w2v.Vocab(None, None, to_dev(counts), None, V, int(counts.sum()), None)
    model = w2v.make_model(syn0, syn1, voc, tree, stride=(dim + 3) // 4 * 4, pad_value=float("nan"))
    p = w2v.Params(window=win, sample=0.0, seed=9, doc_len=doc_len, arch=arch)
    s, n, nodes = w2v.hs_loglik(model, to_dev(tv), p)
    op = oracle.params(V, dim, window=win, sample=0.0, train_words=int(counts.sum()), seed=9, doc_len=doc_len, arch=arch)
    so, no, nodes_o = oracle.loglik(syn0, syn1, otree, tv, op)
    assert (n, nodes) == (no, nodes_o)
    assert abs(s - so) <= (1e-12 if arch == 1 else 1e-6) * abs(so)


# A text of more work units than one launch's wavefronts can number (2^26): its objective is the sum of its halves'.
@pytest.mark.parametrize("kind", ["skip-gram", "cbow", "negative sampling"])
def test_objective_of_more_units_than_a_launch_is_the_sum_of_its_halves(w2v, kind):
    log(f"objective over 2^26 + 10 documents, {kind}")
    V, dim, half = 50, 8, (1 << 26) + 10   # documents of two words: a work unit each
    counts = to_dev(np.arange(V, 0, -1, dtype=np.int64) * 1000)
    tok = torch.randint(V, (2 * half,), generator=torch.Generator(device="cuda").manual_seed(5), device="cuda",
                        dtype=torch.int32)
    voc = w2v.Vocab(None, None, counts, None, V, int(counts.sum()), None)
    syn0, syn1 = synth.init_weights(V, dim, syn1_scale=0.5)
    args = dict(window=1, doc_len=2, seed=4, arch=int(kind == "cbow"), negative=2)
    if kind == "negative sampling":
        model = w2v.make_ns_model(syn0, synth.init_weights(V, dim)[0], voc)
        noise = w2v.build_noise_table(counts)
        run = lambda t, first: w2v.ns_objective(model, noise, t, w2v.Params(first_raw_index=first, **args))
    else:
        model = w2v.make_model(syn0, syn1, voc, w2v.build_huffman(counts))
        run = lambda t, first: w2v.hs_loglik(model, t, w2v.Params(first_raw_index=first, **args))
    whole, a, b = run(tok, 0), run(tok[:half], 0), run(tok[half:], half)
    assert whole[1:] == tuple(x + y for x, y in zip(a[1:], b[1:])) and whole[1] == 2 * half
    # 64-bit sums of 2^27 terms of one sign, in another order
    assert abs(whole[0] - (a[0] + b[0])) <= 1e-10 * abs(whole[0])


# ------------------------------------------------------------- vocabulary
# One tile of the sort and its edges, several, counts of one digit and of more, every id kept and every id dropped;
# the long texts' lists (8 million tokens, ids past 36,864): ids that all go to the lists, which then overflow
# to memory's adds, one id past the bins, a text that is not 16-byte aligned, one of the look-up's size.
@pytest.mark.parametrize("n,ids,kind,min_count,shift", [
    (1, 1, "flat", 1, 0), (700, 4096, "flat", 0, 0), (5000, 4097, "zipf", 2, 1), (300_000, 4096, "zipf", 5, 0),
    (70_000, 8193, "one", 1, 0), (50_000, 3000, "flat", 1000, 0), (8_000_003, 36_865, "zipf", 5, 1),
    (8_000_001, 50_000, "cold", 3, 0), (8_000_000, 300_007, "zipf", 5, 0), (16_000_002, 1_000_003, "zipf", 2, 2),
])
def test_vocab_variants_match_numpy(w2v, n, ids, kind, min_count, shift):
    log(f"vocab n={n} ids={ids} {kind} min_count={min_count} shift={shift}")
    rng = np.random.default_rng(n + ids)
    if kind == "flat":
        tok = rng.integers(0, ids, n + shift)
    elif kind == "one":
        tok = np.where(rng.random(n + shift) < 0.9, ids - 1, rng.integers(0, ids, n + shift))
    elif kind == "cold":
        tok = rng.integers(36_864, ids, n + shift)
    else:
        tok = np.minimum(np.floor(np.exp(rng.random(n + shift) * np.log(ids + 1.0))) - 1, ids - 1)
    tok = tok.astype(np.int32)
    voc = w2v.build_vocab(to_dev(tok)[shift:], ids, min_count)
    tok = tok[shift:]
    counts = np.bincount(tok, minlength=ids)
    order = np.lexsort((np.arange(ids), -counts))
    order = order[counts[order] >= min_count]
    i2v = np.full(ids, -1, np.int32)
    i2v[order] = np.arange(order.size)
    assert (voc.V, voc.train_words) == (order.size, int(counts[order].sum()))
    np.testing.assert_array_equal(voc.counts_by_id.cpu().numpy(), counts)
    np.testing.assert_array_equal(voc.vocab_ids.cpu().numpy(), order)
    np.testing.assert_array_equal(voc.vocab_counts.cpu().numpy(), counts[order])
    np.testing.assert_array_equal(voc.id_to_vocab.cpu().numpy(), i2v)
    np.testing.assert_array_equal(voc.tokens.cpu().numpy(), i2v[tok])


def test_vocab_long_text_out_of_range_token_is_an_error(w2v):
    tok = np.full(8_000_000, 40_000, np.int32)
    tok[7_999_999] = 50_000
    with pytest.raises(w2v.W2VError) as e:
        w2v.build_vocab(to_dev(tok), 50_000, 1)
    assert e.value.code == w2v.W2V_E_RANGE
