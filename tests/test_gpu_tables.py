"""N-gram tables as a parameter of a live context: the storage-saving variant with orders
n = 2..4 only (appendix "Perplexity Evaluation with Fewer N-Grams": same interpolation weights,
alpha = 0.55, tau = 0.1), k up to 10 (the largest k the paper evaluates), and tables replaced
between two timesteps of a generation.  HIP path against the oracle, through the C ABI."""
import numpy as np
import pytest

import synth
from gpu_common import RTOL, compare_step, make_oracle, tails_of, teacher_forced
from oracle import spd_oracle as O

pytestmark = pytest.mark.gpu


def P():
    import paper_2405_18400_amd as pkg
    return pkg


def visits_of(shape, w, prefix, k, n_tokens):
    lm = make_oracle(shape, w)
    _, recs = O.generate(lm, None, prefix, O.DecodeCfg(k, 0.0), n_tokens)
    return [(tuple(rec.state_in.history(i)), int(tok)) for rec in recs[1:] for i in range(k) for tok in rec.top_ids]


@pytest.fixture(scope="module")
def tiny():
    shape = synth.TINY
    w = synth.make_weights(shape, seed=0)
    prefix = synth.make_prefix_uniform(shape.vocab, 16, seed=0)
    return shape, w, prefix


@pytest.mark.parametrize("k", [3, 10])
def test_orders_2_to_4_only(tiny, k):
    shape, w, prefix = tiny
    pkg = P()
    base = synth.make_ngram_tables_zipf(shape.vocab, 40_000, seed=4)
    planted = synth.plant_ngrams(base, visits_of(shape, w, prefix, k, 6), shape.vocab, seed=k)
    small = {n: planted[n] for n in (2, 3, 4)}
    lam = synth.PAPER_LAMBDAS
    sess = pkg.Session(shape, w, max_ctx=64, k_max=16)
    try:
        sess.spd_load_ngrams(small, lam)
        dc = pkg.SpdDecodeCfg(k, 0.55, 0.1, 0.1)
        cfg = O.DecodeCfg(k, 0.55, 0.1, 0.1, tuple(lam))
        _, recs, stats = teacher_forced(sess, make_oracle(shape, w), small, lam, prefix, cfg, 6, RTOL[shape.dtype], dc)
        assert any(c.overlap for r in recs[1:] for c in r.candidates), "planting produced no n-gram hit"
        # the two missing orders change the result: the same run with all five orders differs
        otabs = O.NgramTables(planted)
        _, recs_full = O.generate(make_oracle(shape, w), otabs, prefix, cfg, 6)
        assert any(not np.array_equal(a.pngram, b.pngram) for a, b in zip(recs[1:], recs_full[1:]))
    finally:
        sess.close()


@pytest.mark.parametrize("k", [1, 4, 5, 16])
def test_five_orders_over_the_numbers_of_probes(tiny, k):
    """Up to four drafts the contexts' totals are looked up together with the counts, a group of lanes per probe; from five on
    before them, and the counts four probes to a group; 16 drafts take three rounds of those."""
    shape, w, prefix = tiny
    pkg = P()
    lam = synth.PAPER_LAMBDAS
    tabs = synth.plant_ngrams(synth.make_ngram_tables_zipf(shape.vocab, 40_000, seed=4), visits_of(shape, w, prefix, k, 5), shape.vocab, seed=k)
    sess = pkg.Session(shape, w, max_ctx=64, k_max=16)
    try:
        sess.spd_load_ngrams(tabs, lam)
        cfg = O.DecodeCfg(k, 0.54, 1.0, 0.1, tuple(lam))
        _, recs, _ = teacher_forced(sess, make_oracle(shape, w), tabs, lam, prefix, cfg, 5, RTOL[shape.dtype], pkg.SpdDecodeCfg(k, 0.54, 1.0, 0.1))
        assert any(c.overlap for r in recs[1:] for c in r.candidates), "planting produced no n-gram hit"
    finally:
        sess.close()


@pytest.mark.parametrize("k", [5, 6, 7, 8, 9, 10, 11])
def test_probes_per_group_of_lanes(k):
    """From five drafts on a group of lanes takes one to four probes, by what its wave has left of 5 k^2 (125, 180, 245, 320, 405, 500, and
    605 in two rounds): some waves of a block take one more than others.  From nine drafts on the merge looks at two candidates a
    thread (288 .. 352 of 32 slices).  Scripted logits over tables that most of the probes hit, counts and probabilities without a gap."""
    import torch
    pkg = P()
    shape = synth.ModelShape("one-head", 1, 64, 1, 1, 128, 32000, "fp32")
    rng = np.random.default_rng(k)
    corpus = rng.integers(0, 12, size=4000)
    tabs = {n: np.unique(np.lib.stride_tricks.sliding_window_view(corpus, n), axis=0, return_counts=True) for n in range(2, 7)}
    tabs = {n: (np.ascontiguousarray(keys, np.int32), counts.astype(np.uint32)) for n, (keys, counts) in tabs.items()}
    lam, pre = synth.PAPER_LAMBDAS, corpus[:7].astype(np.int32)
    sess = pkg.Session(shape, synth.make_weights(shape, seed=1), max_ctx=32, k_max=16)
    try:
        sess.spd_load_ngrams(tabs, lam)
        otabs = O.NgramTables(tabs)
        sess.spd_prefill(pre)
        dc, cfg, state, hits = pkg.SpdDecodeCfg(k, 0.54, 1.0, 0.1), O.DecodeCfg(k, 0.54, 1.0, 0.1, lam), None, 0
        for step in range(4):
            z = rng.standard_normal(shape.vocab).astype(np.float32) - 12.0
            z[:12] = rng.permutation(12).astype(np.float32) / 2
            state, rec = O.first_step(z, pre, cfg) if state is None else O.expand_and_prune(state, z, otabs, cfg)
            sess.spd_expand_prune(dc, torch.from_numpy(z).cuda(), first=(step == 0))
            tails, scores, gamma = sess.spd_get_state()
            ids, _, _, valid, png = sess.spd_get_step_info(k)
            assert list(ids) == list(rec.top_ids) and np.array_equal(tails, tails_of(state))
            np.testing.assert_allclose(scores, state.logscores, rtol=1e-5, atol=1e-5)     # sums of fp32 logarithms
            np.testing.assert_allclose(gamma, O.superposition_weights(state.logscores), rtol=1e-4)
            if step > 0:
                np.testing.assert_allclose(png, rec.pngram, rtol=1e-6)                    # five fp32 terms
                hits += int(np.count_nonzero(png))
        assert hits > k * k
    finally:
        sess.close()


def test_tables_replaced_between_timesteps(tiny):
    """Three timesteps with five orders, then the tables are replaced by a different set with
    orders 2..4 on the live context, three more timesteps.  The oracle is driven step by step
    with the same switch."""
    shape, w, prefix = tiny
    pkg = P()
    k, lam = 3, synth.PAPER_LAMBDAS
    visits = visits_of(shape, w, prefix, k, 6)
    tabs_a = synth.plant_ngrams(synth.make_ngram_tables_zipf(shape.vocab, 40_000, seed=5), visits, shape.vocab, seed=1)
    tabs_b = synth.plant_ngrams(synth.make_ngram_tables_zipf(shape.vocab, 30_000, seed=6), visits, shape.vocab, seed=2, frac=0.8)
    tabs_b = {n: tabs_b[n] for n in (2, 3, 4)}
    cfg = O.DecodeCfg(k, 0.54, 1.0, 0.1, tuple(lam))
    dc = pkg.SpdDecodeCfg(k, 0.54, 1.0, 0.1)
    lm = make_oracle(shape, w)
    lm.reset()
    sess = pkg.Session(shape, w, max_ctx=64, k_max=8)
    try:
        sess.spd_load_ngrams(tabs_a, lam)
        sess.spd_prefill(prefix)
        state, rec = O.first_step(lm.forward(lm.embedding_rows(prefix)), prefix, cfg)
        sess.spd_step_outputs = sess.spd_step(dc)
        compare_step(sess, rec, dc, RTOL[shape.dtype], first=True, cfg=cfg, otabs=O.NgramTables(tabs_a), prefix=prefix)
        seen = []
        for t in range(1, 6):
            if t == 3:
                sess.spd_load_ngrams(tabs_b, lam)
            otabs = O.NgramTables(tabs_a if t < 3 else tabs_b)
            gamma = O.superposition_weights(state.logscores)
            x = O.superposed_embedding(lm.embedding_rows([d[-1] for d in state.drafts]), gamma.astype(np.float32))
            sess.spd_set_state(tails_of(state), state.logscores)
            state, rec = O.expand_and_prune(state, lm.forward(x[None, :]), otabs, cfg, gamma_in=gamma)
            sess.spd_step_outputs = sess.spd_step(dc)
            compare_step(sess, rec, dc, RTOL[shape.dtype], first=False, cfg=cfg, otabs=otabs, prefix=prefix)
            seen.append(rec.pngram.copy())
        assert all(np.any(p > 0) for p in seen), "a timestep without any n-gram hit does not test the tables"
    finally:
        sess.close()


@pytest.mark.parametrize("k", [1, 5, 10])
@pytest.mark.parametrize("vocab", [700, 5122, 131072, 131074])
def test_decisions_whose_last_slice_goes_on(vocab, k):
    """One slice, a ragged number of them, the last and the first vocabulary of slices of up to 1024 entries: up to there, with n-grams (five
    drafts and more) and without the same launch selects and decides, timestep after timestep, else the slices have a launch of
    their own: scripted logits, no gap allowance."""
    import torch
    pkg = P()
    shape = synth.ModelShape("one-head", 1, 64, 1, 1, 128, vocab, "fp32")
    rng = np.random.default_rng([vocab, k])
    corpus = rng.integers(0, 40, size=3000)
    tabs = {n: np.unique(np.lib.stride_tricks.sliding_window_view(corpus, n), axis=0, return_counts=True) for n in range(2, 7)}
    tabs = {n: (np.ascontiguousarray(keys, np.int32), counts.astype(np.uint32)) for n, (keys, counts) in tabs.items()}
    lam, pre = synth.PAPER_LAMBDAS, corpus[:7].astype(np.int32)
    sess = pkg.Session(shape, synth.make_weights(shape, seed=1), max_ctx=32, k_max=16)
    try:
        sess.spd_load_ngrams(tabs, lam)
        otabs = O.NgramTables(tabs)
        sess.spd_prefill(pre)
        sess.spd_set_kernel_timing(True)
        for alpha in (0.54, 0.0):
            dc, cfg, state = pkg.SpdDecodeCfg(k, alpha, 1.0, 0.1), O.DecodeCfg(k, alpha, 1.0, 0.1, lam), None
            for step in range(4):
                z = rng.standard_normal(vocab).astype(np.float32) - 12.0
                top = np.concatenate([rng.choice(40, size=12, replace=False), [vocab - 1]])
                z[top] = rng.permutation(len(top)).astype(np.float32) / 2
                state, rec = O.first_step(z, pre, cfg) if state is None else O.expand_and_prune(state, z, otabs, cfg)
                sess.spd_expand_prune(dc, torch.from_numpy(z).cuda(), first=(step == 0))
                tails, scores, _ = sess.spd_get_state()
                assert list(sess.spd_get_step_info(k)[0]) == list(rec.top_ids)
                np.testing.assert_allclose(scores, state.logscores, rtol=1e-5, atol=1e-5)     # sums of fp32 logarithms
                assert np.array_equal(tails, tails_of(state))
        launches = sess.spd_get_kernel_timing()
        assert launches["expand_prune"][1] == 8 and launches["topk_partial"][1] == (8 if vocab > 131072 else 3 if k < 5 else 0)
    finally:
        sess.close()
